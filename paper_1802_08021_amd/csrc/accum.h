// The tile pass of the sparse reduce (kernel k_acc and what it shares with
// the host): included by one source per mode, so that they compile apart.
//
// One workgroup of 16 waves walks a chunk of the index range in tiles of T
// indices.  The P tree slots are cut into NB blocks of consecutive ranks (a
// subtree each), and LDS holds one plane of T values per block.  An entry
// takes its place with one integer LDS atomic, an OR of its block's bit into
// its index's field whose return value tells what was there:
//
//   first of its block   stores its value in the plane;
//   second               adds its value to the first's after a barrier (one
//                        addition is the same in either order);
//   third or later       makes the index "heavy": all its entries are
//                        scattered by rank into a row of P words and the row is
//                        summed as the tree over all P slots.
//
// The root at an index is the tree over the NB planes.  Absent values are
// -0.0, the identity of fp32 addition, so the sum over all slots, present or
// not, rounds exactly as recursive doubling over the ranks present: no node
// bookkeeping is needed for the values.  Collisions inside a block are rare
// by the choice of NB (see acc_blocks), so an entry costs about a dozen
// vector instructions and two LDS operations, and the planes are read once
// in 16-byte pieces.
// (LDS float atomics would need neither the fields nor the second step, but
// ds_add_f32 takes 193 cycles a wave here against 7.4 for an integer one.)
//
// What bounds it: no one thing.  At 128 ranks, 1% of 2^27, a wave takes 300
// vector, 64 scalar and 25 LDS instructions a tile (about fifty a slot) and
// waits 55% of its cycles, for the LDS pipe (a scattered access of a wave takes
// 7 cycles, an entry needs two; half of its cycles are conflicts), the three
// barriers of a tile and memory.  A tile's windows are requested during the one
// before, except where a chunk is a
// tile or two (its first windows), where windows are read on (below), and, above
// 128 slots, where heavy indices ask for entries that were not kept.  The walk it replaced
// ranked every entry among its tile's and merged them index by index.  Whole
// calls, before and after: 128 ranks at 1% of 2^27, 4-bit codes: 1186 -> 810
// us; 64 ranks, zipf supports, 2^26: 298 -> 214 us (heavy indices: half of
// the pass); 24 ragged ranks, sparse root of 5e7: 333 -> 105 us; 128 ranks
// that share one support: 3.9 ms -> 0.17 ms.
//
// Clusters: where more of a stream than its window ends in a tile, the wave
// reads on, up to eight windows in flight, and what needs the entries a second
// time (node sizes, heavy indices) reads those again; heavy indices beyond the
// rows that fit are taken in rounds of consecutive indices, each of which reads
// only its own part.  Runs of 4096 indices that all ranks share, 2^17 entries a
// rank of 2^23: 64 ranks 0.48 ms, 128 ranks 0.95 ms, 256 ranks 2.0 ms (one
// window at a time, all of them again each round: 1.7, 2.9 and 10.3 ms; the
// walk named above: 0.85, 1.7 and 3.6 ms).  An even call pays about 1% for the
// larger code.
//
// Node sizes (INFO): the field is then the mask of all P slots present.  With
// pred the next lower slot present at an entry's index, the two meet in one
// tree node, and |node| = |left| + |right| - the pairs that meet there: one LDS
// histogram over the nodes is all that is counted.
// (Where few indices have two entries, accum_pairs.hip counts them instead.)
#pragma once

#include "internal.h"
#include "qsgd_device.h"

#include <type_traits>

namespace sparcml {

enum AccMode { kAccDense = 0, kAccCount = 1, kAccWrite = 2 };

// How the root's representation is known (AccArgs::when).
enum AccWhen : uint32_t {
    kWhenSparse = 0,  // all sparse: the streams hold at most thr entries together
    kWhenNodes = 1,   // from the node sizes
    kWhenUnion = 2    // from the root's union where it decides, else from the node sizes
};

constexpr uint32_t kVoid = 128;  // two windows

struct AccArgs {
    const StreamDesc* tab;
    const uint32_t* off;   // [P][nchunks + 1] first entry of each chunk
    uint32_t* chunk_ne;    // [nchunks] union size of each chunk
    uint32_t* node_cnt;    // [P - 1] pairs that meet in each node (level order)
    uint32_t* out_idx;
    float* out_val;
    ReduceResult* hdr;     // root header, and the caller's (NULL: none)
    ReduceResult* res;
    uint64_t* node_nnz;
    uint8_t* node_dense;
    const uint32_t* none;    // [kVoid] words 0xFFFFFFFF
    const uint32_t* odd;     // [P] whether a stream is far from even over the chunks
    uint64_t N, thr, chunk;  // range, threshold, indices per chunk (a multiple of 64)
    uint32_t P, L, T;        // tree slots, log2 P, tile width (a multiple of 64)
    uint32_t nchunks, qbits, lo, out_cap, nfold, when;
    uint32_t wshift;         // the chunks' weights (acc_cut) are held shifted down by it, their sum in 31 bits
    uint32_t out_vec;        // out_val is 16-byte aligned
};

// Blocks of a pass with values, by the mean entries per index (of all
// streams together): the fewer, the fewer planes to read and the wider the
// tile; the more, the fewer third arrivals.  Two up to a mean of 0.4 (one
// heavy index in 450), four up to 1.6 (one in 30 at 1.28), else eight.  But
// (2^25 indices, fp32, us):
// - 8 slots: four blocks hold two ranks each, and no index is ever heavy; two up
//   to 0.25 (0.35: 197, with four 115);
// - 16 slots: the wide tile pays up to 1.5 (0.5: 244 with four, 145 with two;
//   0.7 291, 240; 1 313, 288; 1.4 361, 347);
// - above 128 slots a tile's heavy indices cost a second look at 16 slots a
//   wave: two up to 0.5, then eight at once (256 slots, 0.5: 507 with four, 365
//   with two; 0.75 564 with four, 412 with eight; 1 614, 450; 1.4 1086, 544).
inline uint32_t acc_blocks(uint64_t sum_nnz, uint64_t N, uint32_t P)
{
    if (P > 128u) return 2u * sum_nnz <= N ? 2u : 8u;
    if (P == 8u && 4u * sum_nnz > N && 5u * sum_nnz <= 8u * N) return 4u;
    if (P == 16u && 2u * sum_nnz <= 3u * N) return 2u;
    return 5u * sum_nnz <= 2u * N ? 2u : (5u * sum_nnz <= 8u * N ? 4u : 8u);
}
// With node sizes: eight where a quarter of the slots would not fit a mask word.
constexpr uint32_t acc_info_blocks(uint32_t pmax) { return pmax <= 128u ? 4u : 8u; }

// Widest tile: NB planes of T values in 128 KB of LDS, and at four blocks
// 4096 (where the mean entries of a stream rarely ask for more); with node
// sizes the masks of the slots beside them.
constexpr uint32_t acc_tmax(uint32_t nb, bool info, uint32_t pmax)
{
    return !info ? (nb == 2u ? 16384u : 4096u) : (pmax <= 128u ? 4096u : 2048u);
}

// One source each: dense without and with node sizes, counts, sparse output.
hipError_t acc_dense_launch(const AccArgs& a, uint32_t nb, bool info, hipStream_t s);
hipError_t acc_count_launch(const AccArgs& a, bool info, hipStream_t s);
hipError_t acc_write_launch(const AccArgs& a, uint32_t nb, hipStream_t s);
hipError_t acc_pairs_launch(AccArgs a, uint64_t sum_nnz, hipStream_t s);  // node sizes alone (accum_pairs.hip)

#ifdef __HIPCC__
namespace {

// Pointers that live in memory are generic unless marked: generic (FLAT)
// loads also count against the LDS wait counter and would serialize LDS work
// behind every HBM access.
typedef const uint32_t __attribute__((address_space(1))) g_u32;

// Mask of the active lanes where a < b (unsigned), where v is neither zero:
// one compare each.
__device__ __forceinline__ uint64_t lanes_lt(uint32_t a, uint32_t b) { return __builtin_amdgcn_uicmp(a, b, 36); }
__device__ __forceinline__ uint64_t lanes_eq0(uint32_t a) { return __builtin_amdgcn_uicmp(a, 0u, 32); }
__device__ __forceinline__ uint64_t lanes_ne(uint32_t a, uint32_t b) { return __builtin_amdgcn_uicmp(a, b, 33); }
__device__ __forceinline__ uint64_t lanes_nonzero(float v) { return __builtin_amdgcn_fcmpf(v, 0.0f, 14); }
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// base + the number of lanes below this one set in m.
__device__ __forceinline__ uint32_t below_count(uint64_t m, uint32_t base)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}

template <int CTRL>
__device__ __forceinline__ float dpp_plus(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over all 1024 threads.
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* s_tot)
{
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
    const uint32_t s = wave_scan(v);
    __syncthreads();
    if (lane == 63u) s_tot[wv] = s;
    __syncthreads();
    uint32_t t = 0u;
    for (uint32_t w = 0; w < 16u; ++w) t += s_tot[w];
    return t;
}

// The root's representation, in every workgroup alike: the union of the
// chunks, the entries of the chunks before `chunk` (*before), and where the
// node sizes decide, the switch rule level by level (a node is dense iff a
// child is dense or the children's sizes sum past thr; a sparse node's size is
// its children's less the pairs that meet in it).  Workgroup 0 reports the
// header and the nodes.  Returns whether the root is dense.
__device__ bool acc_root(const AccArgs& a, uint32_t chunk, uint32_t* before, uint32_t* s_tot, uint64_t* s_n,
                         uint8_t* s_d, bool report)
{
    const uint32_t t = threadIdx.x;
    uint32_t mine = 0u, pre = 0u;
    for (uint32_t c = t; c < a.nchunks; c += 1024u) {
        const uint32_t n = a.chunk_ne[c];
        mine += n;
        pre += c < chunk ? n : 0u;
    }
    const uint32_t U = block_sum(mine, s_tot);
    *before = block_sum(pre, s_tot);
    bool dense = false;
    uint64_t nnz = U;
    const bool nodes = a.when == kWhenNodes || (a.when == kWhenUnion && U <= a.thr && 2ull * U > a.thr);
    if (a.when == kWhenUnion && U > a.thr) {  // then its children hold more than thr together
        dense = true;
        nnz = a.N;
    }
    if (nodes) {
        __syncthreads();
        if (t < a.P) {
            s_n[t] = a.tab[t].nnz;
            s_d[t] = 0;
        }
        __syncthreads();
        uint32_t node = 0;
        for (uint32_t width = a.P; width > 1u; width >>= 1) {
            bool d = false;
            uint64_t n = 0;
            if (t < width / 2u) {
                const uint64_t both = s_n[2u * t] + s_n[2u * t + 1u];
                d = s_d[2u * t] || s_d[2u * t + 1u] || both > a.thr;
                n = d ? a.N : both - a.node_cnt[node + t];
            }
            __syncthreads();
            if (t < width / 2u) {
                s_n[t] = n;
                s_d[t] = d ? 1 : 0;
                const uint32_t id = node + t;
                // level 1 reports its first nfold nodes, the levels above all
                if (report && (width < a.P || t < a.nfold)) {
                    const uint32_t o = width < a.P ? id - a.P / 2u + a.nfold : t;
                    if (a.node_nnz) a.node_nnz[o] = n;
                    if (a.node_dense) a.node_dense[o] = d ? 1 : 0;
                }
            }
            __syncthreads();
            node += width / 2u;
        }
        dense = s_d[0] != 0;
        nnz = s_n[0];
        __syncthreads();
    }
    if (report && t == 0u) {  // the error words beside them were cleared by the partition launch
        a.hdr->nnz = nnz;
        a.hdr->dense = dense ? 1u : 0u;
        if (a.res) {
            a.res->nnz = nnz;
            a.res->dense = dense ? 1u : 0u;
        }
    }
    return dense;
}

// Where the streams' entries lie unevenly over the chunks, the workgroups take
// ranges of equal weight instead (entries count twice, indices once: a tile's
// cost without entries is about half of what it costs with one an index).  A
// chunk that weighs more than one range is cut into pieces of equal width.
// From the offsets at the chunks, in every workgroup and every pass alike; s_w
// holds 2048 words, s_tot 16.  Returns false where no chunk weighs more than
// 1.5 of the mean.
// (128 ranks, 1% of 2^22 in one layer of a twentieth of the range: 2.3 -> 0.31
// ms; a run that all share: 7.5 -> 0.64 ms.)
__device__ __forceinline__ bool acc_cut(const uint32_t* off, uint32_t P, uint32_t nchunks, uint64_t N, uint64_t chunk,
                                     uint32_t wshift, uint32_t* s_w, uint32_t* s_tot, uint64_t* from, uint64_t* to)
{
    const uint32_t t = threadIdx.x, n = nchunks;
    // four threads a chunk, each a quarter of the streams
    for (uint32_t c0 = 0; c0 < n; c0 += 256u) {
        const uint32_t c = c0 + (t >> 2);
        uint64_t e = 0;
        if (c < n)
            for (uint32_t r = t & 3u; r < P; r += 4u) {
                const uint32_t* const o = off + (uint64_t)r * (n + 1u) + c;
                e += max(o[1], o[0]) - o[0];
            }
        e += __shfl_xor(e, 1);
        e += __shfl_xor(e, 2);
        if (c < n && (t & 3u) == 0u) s_w[c] = (uint32_t)((2u * e + min(chunk, N - c * chunk)) >> wshift);
    }
    __syncthreads();
    const uint32_t w = t < n ? s_w[t] : 0u, incl = wave_scan(w);  // (n <= 1024: a chunk a thread)
    __syncthreads();
    if ((t & 63u) == 63u) s_tot[t >> 6] = incl;
    __syncthreads();
    uint32_t before = incl - w, sum = 0u;
    for (uint32_t v = 0; v < 16u; ++v) {
        if (v < t >> 6) before += s_tot[v];
        sum += s_tot[v];
    }
    if (!__syncthreads_or(2ull * n * w > 3ull * sum + 2u * n)) return false;
    const uint64_t len = min(chunk, N - min((uint64_t)t * chunk, N));
    uint64_t* const s_at = reinterpret_cast<uint64_t*>(s_w);
    if (t < 2u) s_at[t] = N;  // (the last range's end; streams that do not ascend may give others none)
    __syncthreads();
    for (uint32_t i = 0; i < 2u; ++i) {
        const uint64_t at = (uint64_t)(blockIdx.x + i) * sum / n;
        if (at >= before && at - before < w) s_at[i] = ((uint64_t)t * chunk + (at - before) * len / w) & ~63ull;
    }
    __syncthreads();
    *from = s_at[0];
    *to = max(s_at[1], s_at[0]);
    __syncthreads();
    return true;
}

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, uint32_t l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, uint32_t l)
{
    return (uint64_t)lane_u32((uint32_t)(v >> 32), l) << 32 | lane_u32((uint32_t)v, l);
}

// The first entries of SL streams (lane s: stream s's indices ib, of `end`)
// whose index is at least x, each known to lie at pos to past: 64 places at a
// time, of all streams together.
template <int SL>
__device__ __forceinline__ uint32_t find_first(uint64_t ib, uint32_t end, uint32_t pos, uint32_t past, uint32_t x)
{
    const uint32_t lane = threadIdx.x & 63u;
    while (lanes_ne(pos, past)) {
        uint32_t y[SL];
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const uint32_t at = lane_u32(pos, s), n = lane_u32(past, s) - at, step = n / 64u + min(n % 64u, 1u);
            const uint32_t e = at + min(lane * step, n - min(n, 1u));
            y[s] = *reinterpret_cast<g_u32*>(lane_u64(ib, s) + 4ull * min(e, lane_u32(end, s) - 1u));
        }
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const uint32_t at = lane_u32(pos, s), n = lane_u32(past, s) - at, step = n / 64u + min(n % 64u, 1u);
            const uint32_t below = (uint32_t)__popcll(__ballot(lane * step < n && y[s] < x));
            // none below: the first; else past the last of them and at most at the next
            const uint32_t a0 = below ? at + (below - 1u) * step + 1u : at, a1 = below ? at + min(below * step, n) : at;
            pos = lane == (uint32_t)s ? a0 : pos;
            past = lane == (uint32_t)s ? a1 : past;
        }
    }
    return pos;
}

// One entry of a sparse root at position o.  Positions come from the union
// sizes that the counting pass and this one take alike, so for streams that
// ascend o < root nnz <= out_cap; streams that do not can make them disagree,
// and such entries are dropped and reported (bit 1 of the header) instead of
// written past the caller's buffer.
__device__ __forceinline__ void put_sparse(const AccArgs& a, uint32_t o, uint32_t index, float v)
{
    if (o < a.out_cap) {
        a.out_idx[o] = index;
        a.out_val[o] = v;
    } else {
        atomicOr(&a.hdr->pad, 2u);
        if (a.res) atomicOr(&a.res->pad, 2u);
    }
}

// SL: slots per wave (16 SL tree slots at most); NB blocks.  A slot's 64-entry
// window (one entry a lane) is requested during the previous tile.
template <int SL, int NB, int MODE, bool INFO, bool QUANT>
__global__ void __launch_bounds__(1024, 4) k_acc(AccArgs a)
{
    constexpr uint32_t NT = 1024u, NW = 16u, PMAX = 16u * SL, TMAX = acc_tmax(NB, INFO, PMAX), IT = TMAX / 4096u ? TMAX / 4096u : 1u;
    constexpr bool VALS = MODE != kAccCount;
    constexpr uint32_t MW = INFO ? (PMAX + 31u) / 32u : 1u;               // mask words per index (INFO)
    constexpr uint32_t FW = INFO ? TMAX * MW : (NB == 2 ? TMAX / 4u : TMAX);  // field words
    constexpr uint32_t LNB = NB == 8 ? 3u : (NB == 4 ? 2u : 1u);
    constexpr uint32_t LC = VALS ? 128u : 1u;                             // second arrivals a wave keeps per tile
    constexpr uint32_t LW = VALS ? NW * LC + NW * LC / 2u : 1u;           // their words
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    static_assert(NB == 2 || NB == 4 || NB == 8, "fields of 8 or 32 bits");

    __shared__ __align__(16) float s_p[VALS ? NB * TMAX + 64 : 4];  // planes; 64 words that take what is nobody's
    // Fields.  Not INFO: bits [0, NB) blocks present, [NB, 2 NB) blocks whose
    // second arrival came; 8 bits an index at two blocks, else 32.  INFO: the
    // slots present.
    __shared__ __align__(16) uint32_t s_f[FW + 64];  // (64 more, all ones, for lanes without an entry)
    __shared__ __align__(16) uint32_t s_l[LW];
    __shared__ uint32_t s_hb[VALS ? TMAX / 32u : 1u];   // heavy indices
    __shared__ uint32_t s_E[INFO ? PMAX : 1u];          // pairs that meet in each node
    __shared__ uint32_t s_tot[NW];
    __shared__ uint32_t s_heavy[2], s_nh[2];            // by tile parity
    float* const s_lv = reinterpret_cast<float*>(s_l);                     // [NW][LC] values ...
    uint16_t* const s_lj = reinterpret_cast<uint16_t*>(s_l + NW * LC);     // ... and indices of second arrivals

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t P = a.P, T = a.T, chunk = blockIdx.x;
    uint32_t wbase = 0u;  // sparse output: entries before this tile
    if (MODE == kAccWrite) {
        // (the rule's tables take the lists' space: 256 sizes, 256 flags)
        static_assert(!VALS || LW * 4u >= 256u * 9u, "tables of the switch rule");
        if (acc_root(a, chunk, &wbase, s_tot, reinterpret_cast<uint64_t*>(s_l), reinterpret_cast<uint8_t*>(s_l + 512),
                     chunk == 0u))
            return;  // dense: written already
        wbase = __builtin_amdgcn_readfirstlane(wbase);
    }
    if (MODE == kAccCount && INFO && a.when == kWhenUnion) {
        // the node sizes only where the root's union leaves the rule open
        uint32_t mine = 0u;
        for (uint32_t c = tid; c < a.nchunks; c += NT) mine += a.chunk_ne[c];
        const uint32_t U = block_sum(mine, s_tot);
        if (U > a.thr || 2ull * U <= a.thr) return;
        __syncthreads();
    }

    // This wave's slots: ranks wv SL ... wv SL + SL - 1, all in one block.
    const uint32_t r0 = wv * SL;
    const uint32_t b0 = r0 < P ? (a.L >= LNB ? r0 >> (a.L - LNB) : r0 << (LNB - a.L)) : 0u;
    const uint32_t pb = b0 * TMAX;
    const uint32_t lblk = a.L >= LNB ? a.L - LNB : 0u;  // log2 of a block's ranks
    uint32_t first_v = 1u << b0;  // held in a vector register, as the atomics take it
    asm("" : "+v"(first_v));
    const uint32_t first_bit = 1u << b0, second_bit = 1u << (NB + b0);
    // (INFO) the block's ranks within its mask word
    const uint32_t bmask = ((lblk >= 5u ? 0u : 1u << (1u << lblk)) - 1u) << ((r0 & 31u) >> lblk << lblk);
    const uint32_t qlog = a.qbits == 8u ? 3u : (a.qbits == 4u ? 2u : 1u);
    const uint32_t plog = a.qbits == 8u ? 0u : (a.qbits == 4u ? 1u : 2u);
    // Slot s's state sits in lane s: what all slots need is computed for all of
    // them at once, and a wave issues one instruction in four cycles whether
    // it is a vector or a scalar one.
    // An empty slot reads kVoid words that are no index of any tile, and never
    // gets past them.
    uint64_t ib = reinterpret_cast<uint64_t>(a.none), vb = ib;     // index and value (or code) arrays
    uint32_t end = kVoid, pos = 0u, upto = 0u;  // entries; next one, and past the last of this chunk
    float unitv = 0.0f;
    uint32_t odd = 0u;
    for (uint32_t r = lane; r < P; r += 64u) odd |= a.odd[r];
    uint64_t clo = (uint64_t)chunk * a.chunk, chi = min(clo + a.chunk, a.N);  // this workgroup's indices
    if (lane < (uint32_t)SL && r0 + lane < P) {
        const StreamDesc& d = a.tab[r0 + lane];
        if (d.nnz) {
            end = (uint32_t)d.nnz;
            ib = reinterpret_cast<uint64_t>(d.idx);
            vb = reinterpret_cast<uint64_t>(QUANT ? static_cast<const void*>(d.qval) : static_cast<const void*>(d.val));
            const uint32_t* const o = a.off + (r0 + lane) * (a.nchunks + 1u) + chunk;
            pos = min(o[0], end);
            upto = min(max(o[1], pos), end);
        }
        if (QUANT && VALS) unitv = level_unit(*d.qscale, a.qbits);
    }
    if (__builtin_expect(lanes_ne(odd, 0u) != 0u, 0) &&
        acc_cut(a.off, P, a.nchunks, a.N, a.chunk, a.wshift, s_f, s_tot, &clo, &chi)) {
        clo = lane_u64(clo, 0u);
        chi = lane_u64(chi, 0u);
        // The streams' first entries at or past clo, from the chunk it lies in.
        const uint32_t c0 = (uint32_t)min(clo / a.chunk, (uint64_t)a.nchunks - 1u);
        const uint32_t c1 = (uint32_t)min((chi + a.chunk - 1u) / a.chunk, (uint64_t)a.nchunks);
        uint32_t past = pos;
        if (lane < (uint32_t)SL && r0 + lane < P && ib != reinterpret_cast<uint64_t>(a.none)) {
            const uint32_t* const o = a.off + (r0 + lane) * (a.nchunks + 1u);
            pos = min(o[c0], end);
            past = min(max(o[c0 + 1u], pos), end);
            upto = min(max(o[c1], pos), end);
        }
        const uint32_t first = a.lo + (uint32_t)clo;
        pos = find_first<SL>(ib, end, pos, past, first);
        __syncthreads();
    }
    // Whether a window of this chunk can reach past a stream's end (one starts
    // at `upto` at most): the chunk then takes the careful way through its
    // windows.
    const uint32_t edge = __builtin_amdgcn_readfirstlane((int)((uint32_t)lanes_lt(end - upto, 64u) & ((1u << SL) - 1u)));
    for (uint32_t i = tid; i < FW + 64u; i += NT) s_f[i] = i < FW ? 0u : ~0u;
    if (VALS)
        for (uint32_t i = tid; i < TMAX / 32u; i += NT) s_hb[i] = 0u;
    if (INFO)
        for (uint32_t i = tid; i < PMAX; i += NT) s_E[i] = 0u;
    if (tid < 2u) s_heavy[tid] = s_nh[tid] = 0u;

    // Windows: 64 entries of a slot's stream, one a lane.  A window of codes
    // starts at a multiple of the codes in a word, so that a lane's place in
    // its word never changes (entries before the slot's position lie before
    // the tile, and count for nothing).  Codes are loaded as whole words (a
    // byte would be widened at once, and so waited for).
    const uint32_t wlog = plog + 2u;  // log2 of the codes in a word
    const uint32_t wmask = QUANT ? (1u << wlog) - 1u : 0u;
    uint32_t lane4 = 4u * lane, laneo = lane >> wlog << 2;  // (32-bit offsets to scalar bases)
    asm("" : "+v"(lane4), "+v"(laneo));
    const uint32_t laneq = lane << qlog;
    // Near its end (n entries), the entry of a lane is the last one at most,
    // and its code's word starts `back` bytes before its own place, so that it
    // ends in the array (one shorter than a word was copied to one by the
    // partition launch).
    auto last = [&](uint32_t n, uint32_t w) -> uint32_t { return min(w + lane, n - 1u); };
    auto back = [&](uint32_t n, uint32_t e) -> uint32_t {
        const uint32_t bytes = max((n + (1u << plog) - 1u) >> plog, 4u), own = e >> wlog << 2;
        return own - min(own, bytes - 4u);
    };
    // Requests the slots' windows from positions w (a vector; multiples where
    // codes want them) on.  Near a stream's end (careful) only the offsets
    // change, and past it an entry is read and counts for nothing: a load
    // behind a branch would be waited for at its end.
    uint64_t ia, va;
    auto aim = [&](uint32_t w) {
        const uint32_t at = min(w, end - 1u);
        ia = ib + 4ull * at;
        if (VALS) va = QUANT ? vb + 4ull * (at >> wlog) : vb + 4ull * at;
    };
    auto load = [&](uint32_t s, uint32_t ox, uint32_t ov, uint32_t& x, uint32_t& v) {
        x = *reinterpret_cast<g_u32*>(lane_u64(ia, s) + ox);
        v = 0u;
        if (VALS) v = *reinterpret_cast<g_u32*>(lane_u64(va, s) + ov);
    };
    // Slot s's window from position w on, wherever it ends.
    auto load_careful = [&](uint32_t s, uint32_t w, uint32_t& x, uint32_t& v) {
        const uint32_t n = lane_u32(end, s), at = min(w, n - 1u), e = last(n, w);
        x = *reinterpret_cast<g_u32*>(lane_u64(ib, s) + 4ull * at + 4u * (e - at));
        v = 0u;
        if (VALS && !QUANT) v = *reinterpret_cast<g_u32*>(lane_u64(vb, s) + 4ull * at + 4u * (e - at));
        if (VALS && QUANT)
            v = *reinterpret_cast<g_u32*>(lane_u64(vb, s) + 4ull * (at >> wlog) - 4u +
                                          ((e >> wlog << 2) - (at >> wlog << 2) + 4u - back(n, e)));
    };
    auto request_all = [&](uint32_t w, uint32_t* x, uint32_t* v, auto careful) {
        if (!decltype(careful)::value) aim(w);
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            if (decltype(careful)::value) {
                load_careful(s, lane_u32(w, s), x[s], v[s]);
                __builtin_amdgcn_sched_barrier(0);  // (one slot's temporaries at a time)
            } else load(s, lane4, QUANT ? laneo : lane4, x[s], v[s]);
        }
    };
    // A window's entries: index in the tile (kNone past the stream's end) and
    // value -- the fp32 word, or the code times the level unit.  Level 0 gives
    // +0.0 (for a sparse root by an integer zero, which has no sign; for a
    // dense one a zero of either sign is an identity).
    const uint32_t lanes = (32u - a.qbits - laneq) & 31u;  // a code's shift to the word's top
    auto view = [&](uint32_t s, uint32_t w, uint32_t x, uint32_t v, uint32_t tlo, uint32_t& j, float& val, auto careful) {
        uint32_t sh = laneq, up = lanes;  // (a bit field's place is taken modulo 32)
        j = x - tlo;
        if (decltype(careful)::value) {
            const uint32_t n = lane_u32(end, s);
            j = lane < n - w ? j : kNone;
            if (QUANT) {
                const uint32_t e = last(n, w);
                sh = (e << qlog) + 8u * back(n, e);
                up = (32u - a.qbits - sh) & 31u;
            }
        }
        const float un = QUANT ? __uint_as_float(lane_u32(__float_as_uint(unitv), s)) : 0.0f;
        if (!VALS) {
            val = 0.0f;
        } else if (!QUANT) {
            val = __uint_as_float(v);
        } else if (MODE == kAccDense) {
            const float mag = __fmul_rn((float)__builtin_amdgcn_ubfe(v, sh, a.qbits - 1u), un);
            val = __uint_as_float(__float_as_uint(mag) | ((v << up) & 0x80000000u));
        } else {
            const uint32_t code = __builtin_amdgcn_ubfe(v, sh, a.qbits);
            const int m = -(int)(code >> (a.qbits - 1u));
            const int lev = (int)(code & ((1u << (a.qbits - 1u)) - 1u));
            val = __fmul_rn((float)((lev ^ m) - m), un);
        }
    };
    // Field of index j: its word and the bit's place in it.
    auto f_word = [&](uint32_t j) -> uint32_t {
        return INFO ? j * MW + (r0 >> 5) : (NB == 2 ? j >> 2 : j);
    };
    auto f_bits = [&](uint32_t j, uint32_t bits) -> uint32_t {
        return INFO || NB != 2 ? bits : bits << ((j & 3u) * 8u);
    };
    auto mark_heavy = [&](uint32_t j, uint32_t par) {
        atomicOr(&s_hb[j >> 5], 1u << (j & 31u));
        s_heavy[par] = 1u;
    };

    const uint32_t cw = (uint32_t)(chi - clo), ntiles = (uint32_t)(((uint64_t)cw + T - 1u) / T);
    // Output of tile t of the chunk, kept in registers until the next tile's
    // arrivals are done: loads and stores complete in order, so a store shortly
    // before a wait for windows would be waited for as well.
    float4 r4[IT];
    auto store = [&](uint32_t tile) {
        const uint32_t rel = tile * T, TT = min(T, cw - rel);
#pragma unroll
        for (uint32_t it = 0; it < IT; ++it) {
            const uint32_t c = it * 4096u + tid * 4u;
            float* const o = a.out_val + clo + rel + c;
            if (c + 4u <= TT && a.out_vec) {
                store_nt(o, r4[it]);
            } else {
                if (c < TT) o[0] = r4[it].x;
                if (c + 1u < TT) o[1] = r4[it].y;
                if (c + 2u < TT) o[2] = r4[it].z;
                if (c + 3u < TT) o[3] = r4[it].w;
            }
        }
    };

    uint32_t x[SL], v[SL];
    request_all(pos & ~wmask, x, v, std::true_type{});
    uint32_t ne = 0u;  // this thread's non-empty indices
    __syncthreads();

    for (uint32_t tile = 0; tile < ntiles; ++tile) {
        const uint32_t rel = tile * T, TT = min(T, cw - rel), par = tile & 1u;
        const uint32_t tlo = a.lo + (uint32_t)clo + rel;
        // Arrivals.  Lanes without an entry (IN: those with one) aim at words
        // that are nobody's, which is cheaper than to mask them.
        uint32_t lcnt = 0u;  // second arrivals listed by this wave
        auto claim = [&](uint32_t s, uint32_t j, uint64_t IN) -> uint32_t {
            return atomicOr(&s_f[in_mask(IN) ? f_word(j) : FW + lane],
                            f_bits(j, INFO ? 1u << ((r0 + s) & 31u) : first_v));
        };
        auto arrive = [&](uint32_t j, float val, uint32_t old, uint64_t IN) {
            if (!VALS) return;
            const uint32_t seen = INFO ? old & bmask : old & f_bits(j, first_bit);
            const uint64_t FIRST = lanes_eq0(seen);  // (lanes without an entry saw ones)
            s_p[pb + (in_mask(FIRST) ? j : NB * TMAX - pb + lane)] = val;
            // an identity (dense: any zero, whose sign the result drops) need
            // not be added
            const uint64_t NZ = MODE == kAccDense ? lanes_nonzero(val) : lanes_ne(__float_as_uint(val), 0x80000000u);
            uint64_t later = IN & ~FIRST & NZ;
            if (later) {
                if (INFO) {  // the mask tells a third arrival
                    const uint64_t third = later & lanes_ne(seen & (seen - 1u), 0u);
                    if (third && in_mask(third)) mark_heavy(j, par);
                    later &= ~third;
                }
                const uint32_t at = below_count(later, lcnt);
                if (in_mask(later)) {
                    if (at < LC) {
                        s_lv[wv * LC + at] = val;
                        s_lj[wv * LC + at] = (uint16_t)j;
                    } else {
                        mark_heavy(j, par);
                    }
                }
                lcnt += (uint32_t)__popcll(later);
            }
        };
        // The windows' in-tile entries (a prefix, streams ascend).  Up to 8
        // slots a wave keep theirs for the rest of the tile; 16 slots keep only the
        // indices, two a register (0xFFFF: none), or nothing.
        constexpr int G = SL < 8 ? SL : 8;
        constexpr bool KEEP = SL <= 8;
        uint32_t jv[G];
        float vv[G];
        constexpr bool PACK = !KEEP && NB == 8;  // (at two blocks the tile is wide, and its outputs take the registers)
        uint32_t jp[PACK ? SL / 2 : 1];
        const uint32_t win0 = pos & ~wmask;
        uint32_t cnt = 0u, full = 0u;  // entries by slot; slots whose window's last entry lies in the tile
        uint32_t near = edge;
        asm volatile("" : "+s"(near));  // (one tile loop for both ways)
#pragma unroll
        for (int g = 0; g < SL; g += G) {
            uint32_t old[G];
            uint64_t IN[G];
            auto slots = [&](auto careful) {
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    view(g + q, decltype(careful)::value ? lane_u32(win0, g + q) : 0u, x[g + q], v[g + q], tlo, jv[q], vv[q],
                         careful);
                    // (decoded here: moved behind the next requests, it would wait for them)
                    if (VALS) asm volatile("" : "+v"(vv[q]));
                    if (decltype(careful)::value) __builtin_amdgcn_sched_barrier(0);
                    IN[q] = lanes_lt(jv[q], TT);
                    if (PACK) {
                        const uint32_t jj = in_mask(IN[q]) ? jv[q] : 0xFFFFu, h = PACK ? (g + q) / 2 : 0u;
                        jp[h] = q & 1 ? jp[h] | jj << 16 : jj;
                    }
                    asm("v_writelane_b32 %0, %1, %2"
                        : "+v"(cnt) : "s"(__builtin_amdgcn_readfirstlane((int)__popcll(IN[q]))), "n"(g + q));
                }
                if (g + G >= SL) {
                    full = (uint32_t)__builtin_amdgcn_uicmp(cnt + (pos - win0), 64u, 32) & ((1u << SL) - 1u);
                    pos = min(pos + cnt, upto);
                    request_all(pos & ~wmask, x, v, careful);
                }
            };
            if (near) slots(std::true_type{});
            else slots(std::false_type{});
#pragma unroll
            for (int q = 0; q < G; ++q) old[q] = claim(g + q, jv[q], IN[q]);
#pragma unroll
            for (int q = 0; q < G; ++q) arrive(jv[q], vv[q], old[q], IN[q]);
        }
        // More windows of the slots in `mask`, from memory: from a slot's window
        // cur (its lane's; 0: the one at win0) on while they end in this tile, at
        // index jmax at most; cur moves past those.  f(slot, index in tile, value,
        // lanes with an entry of the tile).  `few` (a tile with a window or two more
        // than most): first one window a slot, in turn; then kBatch in flight, of
        // one slot or of as many as are left.
        constexpr uint32_t kLogBatch = IT > 1u || !KEEP ? 2u : 3u, kBatch = 1u << kLogBatch;
        auto walk = [&](uint32_t mask, uint32_t& cur, uint32_t jmax, auto few, auto&& f) {
            auto one = [&](uint32_t s, uint32_t w, uint32_t wx, uint32_t wval) -> bool {
                uint32_t j;
                float val;
                view(s, w, wx, wval, tlo, j, val, std::true_type{});
                const uint64_t in = lanes_lt(j, TT);
                if (in) f(s, j, val, in);
                const bool past = (in >> 63) != 0u && lane_u32(j, 63u) <= jmax;
                if (past) cur += lane == s ? 1u : 0u;
                return past;
            };
            auto window = [&](uint32_t s, uint32_t o) -> uint32_t {
                const uint32_t w0 = lane_u32(win0, s);
                return w0 + min(64u * o, lane_u32(end, s) - w0);
            };
            uint32_t live = decltype(few)::value ? 0u : mask;
            for (uint32_t m = decltype(few)::value ? mask : 0u; m; m &= m - 1u) {
                const uint32_t s = (uint32_t)__builtin_ctz(m), w = window(s, lane_u32(cur, s));
                uint32_t wx, wval;
                load_careful(s, w, wx, wval);
                if (one(s, w, wx, wval)) live |= 1u << s;
            }
            while (__builtin_expect(live != 0u, 0)) {
                const uint32_t m = (uint32_t)__popc(live);
                const uint32_t pl = m == 1u ? kLogBatch : (m == 2u ? kLogBatch - 1u : (m <= 4u ? kLogBatch - 2u : 0u));
                const uint32_t per = (1u << (jmax == kNone ? pl : min(pl, 1u))) - 1u;  // (a round takes one or two)
                // lane u: unit u's slot and window (lane 31 is no slot's: empty)
                uint32_t us = 31u, uw = kVoid, nu = 0u;
#pragma unroll 1
                for (uint32_t rest = live; rest && nu < kBatch; rest &= rest - 1u) {
                    const uint32_t s = (uint32_t)__builtin_ctz(rest), w0 = lane_u32(win0, s);
                    const uint32_t o = 64u * (lane_u32(cur, s) + (lane & per));
                    const bool mine = lane - nu <= per;
                    us = mine ? s : us;
                    uw = mine ? w0 + min(o, lane_u32(end, s) - w0) : uw;
                    nu += per + 1u;
                }
                uint32_t x2[kBatch], v2[kBatch];
#pragma unroll
                for (uint32_t u = 0; u < kBatch; ++u) {
                    if (u >= nu) break;
                    load_careful(lane_u32(us, u), lane_u32(uw, u), x2[u], v2[u]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                nu = __builtin_amdgcn_readfirstlane((int)min(nu, kBatch));
                uint32_t going = __builtin_amdgcn_readfirstlane((int)live);
                asm volatile("" : "+s"(nu), "+s"(going));
#pragma unroll 1
                for (uint32_t u = 0; u < nu; ++u) {  // (one copy of the code: the registers move down)
                    const uint32_t s = lane_u32(us, u);
                    if ((going >> s & 1u) && !one(s, lane_u32(uw, u), x2[0], v2[0])) going &= ~(1u << s);
#pragma unroll
                    for (uint32_t i = 0; i + 1u < kBatch; ++i) {
                        x2[i] = x2[i + 1u];
                        v2[i] = v2[i + 1u];
                    }
                }
                live = going;
            }
        };
        if (__builtin_expect(full != 0u, 0)) {  // the windows are continued
            uint32_t more = 0u, cur = 1u;  // entries found, by slot
            walk(full, cur, kNone, std::true_type{}, [&](uint32_t s, uint32_t j, float val, uint64_t in) {
                more += lane == s ? (uint32_t)__popcll(in) : 0u;
                arrive(j, val, claim(s, j, in), in);
            });
            cnt += more;
            pos = min(pos + more, upto);
            // (every slot, in the order above: a wait for one of them then
            // means the same whichever way it was requested)
            request_all(pos & ~wmask, x, v, std::true_type{});
        }
        // Second arrivals of this wave, one or two a lane: kept for the
        // addition behind the barrier unless the index's block already had one.
        uint32_t kj0 = kNone, kj1 = kNone;
        float kv0 = 0.0f, kv1 = 0.0f;
        if (VALS && lcnt) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const uint32_t lc = min(lcnt, LC);
            auto take = [&](uint32_t i, uint32_t& kj, float& kv) {
                if (i < lc) {
                    const uint32_t j = s_lj[wv * LC + i];
                    kv = s_lv[wv * LC + i];
                    kj = j;
                    if (!INFO) {
                        const uint32_t bit = f_bits(j, second_bit);
                        if (atomicOr(&s_f[f_word(j)], bit) & bit) {
                            mark_heavy(j, par);
                            kj = kNone;
                        }
                    }
                }
            };
            take(lane, kj0, kv0);
            if (lc > 64u) take(lane + 64u, kj1, kv1);
        }
        if (MODE == kAccDense && tile != 0u) store(tile - 1u);
        __syncthreads();

        // The wave's entries in this tile once more, at index jmax at most (of
        // those read again, from window cur on): f(slot, index in tile, value).
        // Without the values kept, the windows are read again of the slots that
        // have an entry where(index) wants it; without the indices, of all.
        constexpr uint32_t kCur = KEEP ? 1u : 0u;
        auto kept = [&](int s) -> uint32_t { return KEEP ? jv[KEEP ? s : 0] : jp[PACK ? s / 2 : 0] >> (16 * (s & 1)) & 0xFFFFu; };
        auto again = [&](uint32_t& cur, uint32_t jmax, auto few, auto&& where, auto&& f) {
            uint32_t in = __builtin_amdgcn_readfirstlane((int)TT), reread = full;
            asm volatile("" : "+s"(in));  // (compared anew: eight masks kept over the rounds would not fit the registers)
            if (KEEP) {
#pragma unroll
                for (int s = 0; s < G; ++s)
                    if (jv[s] < in) f((uint32_t)s, jv[s], vv[s]);
            } else if (!PACK) {
                reread = (uint32_t)__builtin_amdgcn_uicmp(cnt, 0u, 33) & ((1u << SL) - 1u);
            } else {
#pragma unroll
                for (int s = 0; s < SL; ++s) {
                    const uint32_t j = kept(s);
                    bool hit = false;
                    if (j < in) hit = where(j);
                    if (__ballot(hit)) reread |= 1u << s;
                }
            }
            walk(reread, cur, jmax, few, [&](uint32_t s, uint32_t j, float val, uint64_t) {
                if (j < in) f(s, j, val);
            });
        };
        if (INFO) {
            static_assert(!INFO || KEEP || PACK, "indices kept");
            // each entry and the next lower slot present at its index meet in a
            // node of level h + 1, h their highest differing bit
            auto meet = [&](uint32_t sl, uint32_t j) {
                const uint32_t r = r0 + sl;
                uint32_t pred = kNone;
#pragma unroll
                for (uint32_t w = 0; w < MW; ++w) {
                    if (w > (r0 >> 5)) break;
                    const uint32_t m = s_f[j * MW + w] & (w == (r0 >> 5) ? (1u << (r & 31u)) - 1u : ~0u);
                    pred = m ? w * 32u + 31u - (uint32_t)__clz(m) : pred;
                }
                if (pred != kNone) {
                    const uint32_t h = 31u - (uint32_t)__clz(pred ^ r);
                    atomicAdd(&s_E[P - (P >> h) + (r >> (h + 1u))], 1u);
                }
            };
#pragma unroll
            for (int s = 0; s < SL; ++s)
                if (kept(s) < TT) meet((uint32_t)s, kept(s));
            uint32_t cur = 1u;
            walk(full, cur, kNone, std::true_type{}, [&](uint32_t s, uint32_t j, float, uint64_t) {
                if (j < TT) meet(s, j);
            });
        }
        if (VALS) {
            if (kj0 != kNone) s_p[pb + kj0] += kv0;
            if (kj1 != kNone) s_p[pb + kj1] += kv1;
        }
        // (the masks read above are cleared below)
        if (VALS || INFO) __syncthreads();
        if (VALS && tid == 0u) s_heavy[par ^ 1u] = s_nh[par ^ 1u] = 0u;

        // Four consecutive indices: the blocks present in each, clearing the
        // fields (bit `top(b)` of word `word(b)` of an index's marks); the tree
        // over the planes.
        constexpr uint32_t CL = SL == 1 ? 4u : (SL == 2 ? 5u : (SL == 4 ? 6u : (SL == 8 ? 7u : 8u)));  // SL > 1: log2 P
        constexpr uint32_t CB = CL - LNB;                                       // and of a block's slots
        constexpr bool WIDE = INFO && SL > 1;
        constexpr uint32_t BW = 1u << (CB < 5u ? CB : 5u);
        constexpr uint32_t HB = BW == 32u ? 0x80000000u : (BW == 16u ? 0x80008000u : (BW == 8u ? 0x80808080u : 0x88888888u));
        static_assert(!WIDE || (CB <= 5u && BW >= 4u), "a block lies in one mask word");
        constexpr uint32_t KW = WIDE ? MW : 1u;
        auto blocks4 = [&](uint32_t c, uint32_t (*pr)[KW]) {
            if (WIDE) {
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i)
#pragma unroll
                    for (uint32_t w = 0; w < MW; ++w) {
                        const uint32_t q = s_f[(c + i) * MW + w];
                        s_f[(c + i) * MW + w] = 0u;
                        // the top bit of each block's field: some slot is present
                        pr[i][w] = (((q & ~HB) + ~HB) | q) & HB;
                    }
            } else if (INFO) {
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) {
                    const uint32_t q = s_f[c + i];
                    s_f[c + i] = 0u;
                    uint32_t m = 0u;
#pragma unroll
                    for (uint32_t b = 0; b < (uint32_t)NB; ++b) {
                        const uint32_t lo = a.L >= LNB ? b << lblk : b >> (LNB - a.L);
                        const uint32_t bm = ((1u << (1u << lblk)) - 1u) << lo;
                        const bool here = a.L >= LNB || (b & ((1u << (LNB - a.L)) - 1u)) == 0u;
                        if (here && (q & bm)) m |= 1u << b;
                    }
                    pr[i][0] = m;
                }
            } else if (NB != 2) {
                const uint4 q = *reinterpret_cast<const uint4*>(&s_f[c]);
                *reinterpret_cast<uint4*>(&s_f[c]) = make_uint4(0u, 0u, 0u, 0u);
                constexpr uint32_t M = (1u << NB) - 1u;
                pr[0][0] = q.x & M;
                pr[1][0] = q.y & M;
                pr[2][0] = q.z & M;
                pr[3][0] = q.w & M;
            } else {
                const uint32_t q = s_f[c >> 2];
                s_f[c >> 2] = 0u;
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) pr[i][0] = (q >> (8u * i)) & 3u;
            }
        };
        auto some = [&](const uint32_t* m) -> uint32_t {
            uint32_t o = m[0];
#pragma unroll
            for (uint32_t w = 1; w < KW; ++w) o |= m[w];
            return min(o, 1u);
        };
        auto planes4 = [&](uint32_t c, uint32_t (*pr)[KW], float* o) {
            constexpr int HALF = NB == 8 ? 4 : NB;  // four planes at a time: eight would not fit the registers
            float half[4];
#pragma unroll
            for (int b0 = 0; b0 < NB; b0 += HALF) {
                float4 p[HALF];
#pragma unroll
                for (int b = 0; b < HALF; ++b) p[b] = *reinterpret_cast<const float4*>(&s_p[(b0 + b) * TMAX + c]);
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) {
                    float t[HALF];
#pragma unroll
                    for (int b = 0; b < HALF; ++b) {
                        const float y = i == 0u ? p[b].x : (i == 1u ? p[b].y : (i == 2u ? p[b].z : p[b].w));
                        const uint32_t w = WIDE ? ((uint32_t)(b0 + b) << CB) >> 5 : 0u;
                        const uint32_t top = WIDE ? (((uint32_t)(b0 + b) << CB) & 31u) + BW - 1u : (uint32_t)(b0 + b);
                        const uint32_t m = (uint32_t)((int)(pr[i][w] << (31u - top)) >> 31);  // all ones: present
                        t[b] = __uint_as_float((__float_as_uint(y) & m) | (0x80000000u & ~m));
                    }
#pragma unroll
                    for (int h = 1; h < HALF; h <<= 1)
#pragma unroll
                        for (int b = 0; b < HALF; b += 2 * h) t[b] = t[b] + t[b + h];
                    if (b0 == 0) half[i] = t[0];
                    o[i] = b0 == 0 ? t[0] : half[i] + t[0];
                }
                if (NB == 8 && b0 == 0) __builtin_amdgcn_sched_barrier(0);
            }
        };
        // This thread's indices: four from own(it) on, it < IT.  (Sparse output
        // needs its entries in index order: wave w takes the w-th sixteenth of
        // the tile, in groups of 256.)
        const uint32_t tw = (T / 16u + 255u) & ~255u, w0 = wv * tw;
        auto own = [&](uint32_t it) -> uint32_t {
            return MODE == kAccWrite ? w0 + it * 256u + lane * 4u : it * 4096u + tid * 4u;
        };
        auto owned = [&](uint32_t it) -> bool { return (MODE != kAccWrite || it * 256u < tw) && own(it) < T; };
        float o[4 * IT];
        uint32_t pk = 0u;  // sparse output: which of them are present
#pragma unroll
        for (uint32_t it = 0; it < IT; ++it) {
            if (!owned(it)) continue;
            uint32_t pr[4][KW];
            blocks4(own(it), pr);
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) {
                if (MODE == kAccWrite) pk |= some(pr[i]) << (4u * it + i);
                else ne += some(pr[i]);
            }
            if (VALS) planes4(own(it), pr, o + 4 * it);
        }
        if (VALS && s_heavy[par]) {
            // Heavy indices, in the planes' space: the owners number them (s_num,
            // kNoNum for the others); rows of P words are cleared, filled by
            // rank and summed into s_out, from where the owners take the sums.
            // Where there are more than rows, they are numbered in index order and
            // taken in rounds: each an interval of the tile, so that of the
            // entries read again a round takes its own part.
            auto ownedh = [&](uint32_t it) -> bool {
                uint32_t t = __builtin_amdgcn_readfirstlane((int)T);
                if (MODE != kAccWrite) asm volatile("" : "+s"(t));  // (as above)
                return (MODE != kAccWrite || it * 256u < tw) && own(it) < t;
            };
            constexpr uint32_t kNoNum = 0xFFFFu;
            float* const s_out = s_p;                                        // [T]
            uint16_t* const s_num = reinterpret_cast<uint16_t*>(s_p + T);    // [T]
            float* const s_row = s_p + T + T / 2u;
            uint16_t* const s_hj = s_lj;                                     // [NW LC] a round's indices
            const uint32_t lg = max(P, 4u) / 4u;                             // lanes per row, four slots each
            const uint32_t RS = 4u * lg + 4u;                                // row words (the rows of a slot on several banks)
            const uint32_t HR = min(min((NB * TMAX - T - T / 2u) / RS, NW * LC), kNoNum);
            uint32_t hm = 0u;  // this thread's
#pragma unroll
            for (uint32_t it = 0; it < IT; ++it)
                if (ownedh(it)) hm |= ((s_hb[own(it) >> 5] >> (own(it) & 31u)) & 15u) << (4u * it);
            const uint32_t hn = (uint32_t)__popc(hm), hs = wave_scan(hn);
            uint32_t first = 0u;
            if (lane == 63u && hs) first = atomicAdd(&s_nh[par], hs);
            first = lane_u32(first, 63u) + hs - hn;
            __syncthreads();
            const uint32_t nh = s_nh[par];
#pragma unroll
            for (uint32_t it = 0; it < IT; ++it) {
                if (!ownedh(it)) continue;
                *reinterpret_cast<uint2*>(&s_num[own(it)]) = make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);
            }
            for (uint32_t i = tid; i < TMAX / 32u; i += NT) s_hb[i] = 0u;
            auto number = [&](uint32_t m, uint32_t id, uint32_t nr) {
                for (; m; m &= m - 1u, ++id) {
                    const uint32_t q = (uint32_t)__builtin_ctz(m), j = own(q >> 2) + (q & 3u);
                    s_num[j] = (uint16_t)(id < nr ? id : kNoNum);
                    if (id < nr) s_hj[id] = (uint16_t)j;
                }
            };
            auto clear_rows = [&](uint32_t nr) {
                for (uint32_t i = tid * 4u; i < nr * RS; i += NT * 4u)
                    *reinterpret_cast<float4*>(&s_row[i]) = make_float4(-0.0f, -0.0f, -0.0f, -0.0f);
                __syncthreads();
            };
            auto scatter = [&](uint32_t& cur, uint32_t jmax, auto few) {
                again(cur, jmax, few, [&](uint32_t j) { return s_num[j] != kNoNum; }, [&](uint32_t sl, uint32_t j, float val) {
                    const uint32_t i = s_num[j];
                    if (i != kNoNum) s_row[i * RS + r0 + sl] = val;
                });
                __syncthreads();
            };
            auto sum_rows = [&](uint32_t nr) {
                const uint32_t rpw = 64u / lg, sub = lane / lg, q4 = (lane % lg) * 4u;  // lg: a power of two
                for (uint32_t i0 = wv * rpw; i0 < nr; i0 += NW * rpw) {
                    const uint32_t i = min(i0 + sub, nr - 1u), j = s_hj[i];
                    const float4 q = *reinterpret_cast<const float4*>(&s_row[i * RS + q4]);
                    float t = (q.x + q.y) + (q.z + q.w);
                    if (lg >= 2u) t = dpp_plus<0xB1>(t);   // lane ^ 1
                    if (lg >= 4u) t = dpp_plus<0x4E>(t);   // lane ^ 2
                    if (lg >= 8u) t = dpp_plus<0x141>(t);  // the other half of 8
                    if (lg >= 16u) t = dpp_plus<0x140>(t); // the other half of 16
                    if (lg >= 32u) t += __shfl_xor(t, 16);
                    if (lg >= 64u) t += __shfl_xor(t, 32);
                    if (q4 == 0u && i0 + sub < nr) s_out[j] = t;
                }
                __syncthreads();
            };
            uint32_t cur = kCur;
            if (__builtin_expect(nh <= HR, 1)) {
                number(hm, first, nh);
                clear_rows(nh);
                scatter(cur, kNone, std::integral_constant<bool, KEEP>{});
                sum_rows(nh);
            } else {
                static_assert(IT * NW <= 64u, "a lane for each wave's 256 indices");
                uint32_t* const s_ht = s_l;  // their counts, in index order
                auto part = [&](uint32_t it) -> uint32_t { return MODE == kAccWrite ? wv * IT + it : it * NW + wv; };
                uint32_t id0[IT];  // the number of the first of four
#pragma unroll
                for (uint32_t it = 0; it < IT; ++it) {
                    const uint32_t n = (uint32_t)__popc(hm >> (4u * it) & 15u), incl = wave_scan(n);
                    if (lane == 63u) s_ht[part(it)] = incl;
                    id0[it] = incl - n;
                }
                __syncthreads();
                const uint32_t ht = lane < IT * NW ? s_ht[lane] : 0u, ps = wave_scan(ht) - ht;
#pragma unroll
                for (uint32_t it = 0; it < IT; ++it) id0[it] += lane_u32(ps, part(it));
#pragma unroll 1
                for (uint32_t base = 0; base < nh; base += HR) {
                    const uint32_t nr = min(nh - base, HR);
#pragma unroll
                    for (uint32_t it = 0; it < IT; ++it) number(hm & 15u << (4u * it), id0[it] - base, nr);
                    clear_rows(nr);
                    scatter(cur, __builtin_amdgcn_readfirstlane((int)s_hj[nr - 1u]), std::false_type{});
                    sum_rows(nr);
                }
            }
#pragma unroll
            for (uint32_t it = 0; it < IT; ++it) {
                if (!ownedh(it)) continue;
                const uint32_t b = hm >> (4u * it) & 15u;
                if (b) {
                    const float4 q = *reinterpret_cast<const float4*>(&s_out[own(it)]);
                    o[4 * it] = b & 1u ? q.x : o[4 * it];
                    o[4 * it + 1] = b & 2u ? q.y : o[4 * it + 1];
                    o[4 * it + 2] = b & 4u ? q.z : o[4 * it + 2];
                    o[4 * it + 3] = b & 8u ? q.w : o[4 * it + 3];
                }
            }
        }
        if (MODE == kAccDense) {
#pragma unroll
            for (uint32_t it = 0; it < IT; ++it)
                r4[it] = make_float4(o[4 * it] + 0.0f, o[4 * it + 1] + 0.0f, o[4 * it + 2] + 0.0f, o[4 * it + 3] + 0.0f);
        }
        if (MODE == kAccWrite) {
            uint32_t nw = 0u, run[IT];  // entries of the wave; this thread's places in them
#pragma unroll
            for (uint32_t it = 0; it < IT; ++it) {
                const uint32_t n = (uint32_t)__popc(pk >> (4u * it) & 15u);
                const uint32_t incl = wave_scan(n);
                run[it] = nw + incl - n;
                nw += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            }
            if (lane == 0u) s_tot[wv] = nw;
            __syncthreads();
            const uint32_t wt = lane < NW ? s_tot[lane] : 0u;
            const uint32_t xs = wave_scan(wt);
            const uint32_t wpre = (uint32_t)__builtin_amdgcn_readlane((int)(xs - wt), (int)wv);
            // through the planes' space, so that the stores are whole lines (24
            // ragged ranks, 5e7 indices: 107 -> 103 us)
            uint32_t* const s_oi = reinterpret_cast<uint32_t*>(s_p) + TMAX;
#pragma unroll
            for (uint32_t it = 0; it < IT; ++it) {
                uint32_t at = wpre + run[it];
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) {
                    if (pk >> (4u * it + i) & 1u) {
                        s_p[at] = o[4 * it + i];
                        s_oi[at++] = tlo + own(it) + i;
                    }
                }
            }
            const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)xs, 63);
            __syncthreads();
            for (uint32_t i = tid; i < all; i += NT) put_sparse(a, wbase + i, s_oi[i], s_p[i]);
            wbase += all;
        }
        __syncthreads();
    }
    if (MODE == kAccDense && ntiles != 0u) store(ntiles - 1u);
    if (MODE != kAccWrite) {
        const uint32_t all = block_sum(ne, s_tot);
        if (tid == 0u) a.chunk_ne[chunk] = all;
    }
    if (INFO) {
        for (uint32_t i = tid; i + 1u < P; i += NT)
            if (s_E[i]) atomicAdd(&a.node_cnt[i], s_E[i]);
    }
}

template <int SL, int NB, int MODE, bool INFO, bool QUANT>
hipError_t acc_launch(const AccArgs& a, hipStream_t s)
{
    const int slot = MODE == kAccWrite ? kTReduceWrite : (MODE == kAccCount && a.when == kWhenUnion ? kTReduceSlow : kTReducePass);
    timer_begin(slot, s);
    hipLaunchKernelGGL((k_acc<SL, NB, MODE, INFO, QUANT>), dim3(a.nchunks), dim3(1024), 0, s, a);
    timer_end(slot, s);
    return hipGetLastError();
}

template <int NB, int MODE, bool INFO, bool QUANT>
hipError_t acc_launch_p(const AccArgs& a, hipStream_t s)
{
    if (a.P <= 16u) return acc_launch<1, INFO ? acc_info_blocks(16) : NB, MODE, INFO, QUANT>(a, s);
    if (a.P <= 32u) return acc_launch<2, INFO ? acc_info_blocks(32) : NB, MODE, INFO, QUANT>(a, s);
    if (a.P <= 64u) return acc_launch<4, INFO ? acc_info_blocks(64) : NB, MODE, INFO, QUANT>(a, s);
    if (a.P <= 128u) return acc_launch<8, INFO ? acc_info_blocks(128) : NB, MODE, INFO, QUANT>(a, s);
    return acc_launch<16, INFO ? acc_info_blocks(256) : (NB == 4 ? 8 : NB), MODE, INFO, QUANT>(a, s);
}

}  // namespace
#endif  // __HIPCC__

}  // namespace sparcml
