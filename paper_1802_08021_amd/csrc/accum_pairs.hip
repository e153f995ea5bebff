// The tree's node sizes, and the union size of every chunk, from the indices
// alone: the pass for streams that rarely meet.
//
// A node's size is its children's less the pairs that meet in it (accum.h), so
// only indices that two ranks or more hold count for anything.  Two bits an
// index in LDS tell which these are: an entry that finds its first bit set sets
// the second.  Then they are numbered, and the streams read once more: an entry
// at one of them sets its rank's bit in the index's row, and each row's
// neighbouring ranks are its pairs.  Up to 2^17 indices a tile, so that a stream
// has many windows in it and their loads are in flight together, whatever the
// number of ranks.  (The tile pass with node sizes holds a mask of all ranks for
// every index: tiles of 2048 or 4096, in which it visits every rank for a few
// entries.)
//
// What bounds it: the two walks, about 40 instructions and three LDS operations
// a window and walk.  Whole calls with node sizes, 2^25 indices, in the tile pass
// and so: 256 ranks at a mean of 0.1 entries an index 1.17 -> 0.23 ms, at 0.5 1.87
// -> 0.69 ms, 128 ranks at 0.25 0.25 -> 0.13 ms, 2 ranks at 0.25 0.29 -> 0.19 ms.
#include "accum.h"

#include <cmath>

namespace sparcml {
namespace {

constexpr uint32_t kPairTile = 1u << 17;          // indices a tile at most
constexpr uint32_t kPairRowWords = 25600;         // rows: 100 KB beside 32 KB of bits and 16 KB of counts
constexpr uint32_t pair_rows(uint32_t mw) { return kPairRowWords / mw; }

// SL slots a wave (16 SL tree slots); with SL = 1 a slot's entries are shared by
// 16 / P waves.
template <int SL>
__global__ void __launch_bounds__(1024, 4) k_pairs(AccArgs a)
{
    constexpr uint32_t NT = 1024u, W = kPairTile / 32u, MW = (16u * SL + 31u) / 32u, R = pair_rows(MW);
    constexpr int GS = SL < 8 ? (SL < 4 ? SL : 4) : 8, U = 8 / GS;  // slots and windows of each in flight
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    __shared__ __align__(16) uint32_t s_once[W + 64], s_twice[W];  // (64 more for lanes without an entry)
    __shared__ __align__(16) uint32_t s_row[kPairRowWords];
    // Counts of the nodes, sixteen copies: lanes that add to one node at once
    // (runs that all ranks share) would wait for each other, as would lanes whose
    // bits lie in one word: consecutive indices take consecutive words.  (16 ranks
    // that share a run, 2^22: 193 -> 160 us a call.)
    constexpr uint32_t EW = 16u * SL + 1u;
    __shared__ uint32_t s_E[16u * EW], s_tot[16];
    static_assert(W == 4096u && kPairTile == 32u * W, "an index's word its low 12 bits, its bit the five above");
    auto word = [](uint32_t j) -> uint32_t { return j & (W - 1u); };
    auto bit = [](uint32_t j) -> uint32_t { return j >> 12 & 31u; };
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t P = a.P, T = a.T, chunk = blockIdx.x;
    if (a.when == kWhenUnion) {  // only where the root's union leaves the rule open
        uint32_t mine = 0u;
        for (uint32_t c = tid; c < a.nchunks; c += NT) mine += a.chunk_ne[c];
        const uint32_t U0 = block_sum(mine, s_tot);
        if (U0 > a.thr || 2ull * U0 <= a.thr) return;
        __syncthreads();
    }
    uint32_t wlog = 0u;  // log2 of the waves a slot
    while (SL == 1 && (P << wlog) < 16u) ++wlog;
    const uint32_t r0 = (wv >> wlog) * SL, part = wv & ((1u << wlog) - 1u);
    uint64_t ib = reinterpret_cast<uint64_t>(a.none);
    uint32_t end = kVoid, pos = 0u, upto = 0u, odd = 0u;
    for (uint32_t r = lane; r < P; r += 64u) odd |= a.odd[r];
    uint64_t clo = (uint64_t)chunk * a.chunk, chi = min(clo + a.chunk, a.N);
    const bool has = lane < (uint32_t)SL && r0 + lane < P && a.tab[r0 + lane].nnz;
    const uint32_t* const off = a.off + (r0 + lane) * (a.nchunks + 1u);
    if (has) {
        const StreamDesc& d = a.tab[r0 + lane];
        end = (uint32_t)d.nnz;
        ib = reinterpret_cast<uint64_t>(d.idx);
        pos = min(off[chunk], end);
        upto = min(max(off[chunk + 1u], pos), end);
    }
    if (__builtin_expect(lanes_ne(odd, 0u) != 0u, 0) &&
        acc_cut(a.off, P, a.nchunks, a.N, a.chunk, a.wshift, s_row, s_tot, &clo, &chi)) {
        clo = lane_u64(clo, 0u);
        chi = lane_u64(chi, 0u);
        const uint32_t c0 = (uint32_t)min(clo / a.chunk, (uint64_t)a.nchunks - 1u);
        const uint32_t c1 = (uint32_t)min((chi + a.chunk - 1u) / a.chunk, (uint64_t)a.nchunks);
        uint32_t past = pos;
        if (has) {
            pos = min(off[c0], end);
            past = min(max(off[c0 + 1u], pos), end);
            upto = min(max(off[c1], pos), end);
        }
        pos = find_first<SL>(ib, end, pos, past, a.lo + (uint32_t)clo);
        upto = max(upto, pos);
    }
    for (uint32_t i = tid; i < W; i += NT) s_once[i] = s_twice[i] = 0u;
    for (uint32_t i = tid; i < 16u * EW; i += NT) s_E[i] = 0u;
    __syncthreads();

    const uint32_t cw = (uint32_t)(chi - clo);
    uint32_t ne = 0u;
    for (uint32_t rel = 0; rel < cw; rel += min(T, cw - rel)) {
        const uint32_t TT = min(T, cw - rel), tlo = a.lo + (uint32_t)clo + rel;
        const uint32_t till = rel + TT < cw ? find_first<SL>(ib, end, pos, upto, tlo + TT) : upto;
        // This wave's entries of the tile, eight windows together: f(indices in
        // the tile (kNone: no entry), their ranks).
        auto each = [&](auto&& f) {
#pragma unroll
            for (int g = 0; g < SL; g += GS) {
                uint32_t at[GS], to[GS], most = 0u;
#pragma unroll
                for (int q = 0; q < GS; ++q) {
                    const uint32_t p0 = lane_u32(pos, g + q), n = lane_u32(till, g + q) - p0;
                    at[q] = p0 + (uint32_t)((uint64_t)n * part >> wlog);
                    to[q] = p0 + (uint32_t)((uint64_t)n * (part + 1u) >> wlog);
                    most = max(most, to[q] - at[q]);
                }
                for (uint32_t o = 0; o < most; o += 64u * U) {
                    uint32_t j[GS * U];
#pragma unroll
                    for (int q = 0; q < GS; ++q)
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint32_t e = at[q] + min(o + 64u * u + lane, to[q] - at[q]);
                            j[q * U + u] = *reinterpret_cast<g_u32*>(lane_u64(ib, g + q) + 4ull * min(e, lane_u32(end, g + q) - 1u));
                        }
#pragma unroll
                    for (int q = 0; q < GS; ++q)
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint32_t i = j[q * U + u] - tlo;
                            j[q * U + u] = o + 64u * u + lane < to[q] - at[q] && i < TT ? i : kNone;
                        }
                    f(j, r0 + g);
                }
            }
        };
        each([&](const uint32_t* j, uint32_t) {
            uint32_t old[GS * U];
#pragma unroll
            for (int k = 0; k < GS * U; ++k)
                old[k] = atomicOr(&s_once[j[k] != kNone ? word(j[k]) : W + lane], 1u << bit(j[k]));
#pragma unroll
            for (int k = 0; k < GS * U; ++k)
                if (j[k] != kNone && (old[k] >> bit(j[k]) & 1u)) atomicOr(&s_twice[word(j[k])], 1u << bit(j[k]));
        });
        __syncthreads();
        // Numbers: s_once takes the first of each word.
        uint32_t nm;
        {
            constexpr uint32_t PER = W / NT;
            const uint4 o4 = reinterpret_cast<const uint4*>(s_once)[tid], t4 = reinterpret_cast<const uint4*>(s_twice)[tid];
            static_assert(PER == 4u, "four words a thread");
            ne += (uint32_t)(__popc(o4.x) + __popc(o4.y) + __popc(o4.z) + __popc(o4.w));
            const uint32_t n0 = (uint32_t)__popc(t4.x), n1 = n0 + (uint32_t)__popc(t4.y), n2 = n1 + (uint32_t)__popc(t4.z);
            const uint32_t n = n2 + (uint32_t)__popc(t4.w), incl = wave_scan(n);
            if (lane == 63u) s_tot[wv] = incl;
            __syncthreads();
            const uint32_t wt = lane < 16u ? s_tot[lane] : 0u, ws = wave_scan(wt);
            nm = lane_u32(ws, 63u);
            const uint32_t first = lane_u32(ws - wt, wv) + incl - n;
            reinterpret_cast<uint4*>(s_once)[tid] = make_uint4(first, first + n0, first + n1, first + n2);
        }
        for (uint32_t base = 0; base < nm; base += R) {
            const uint32_t nr = min(nm - base, R);
            for (uint32_t i = tid; i < nr * MW; i += NT) s_row[i] = 0u;
            __syncthreads();
            each([&](const uint32_t* j, uint32_t r) {
                uint32_t tw[GS * U], id[GS * U];
#pragma unroll
                for (int k = 0; k < GS * U; ++k) {
                    const uint32_t w = j[k] != kNone ? word(j[k]) : 0u;
                    tw[k] = s_twice[w];
                    id[k] = s_once[w];
                }
#pragma unroll
                for (int k = 0; k < GS * U; ++k) {
                    const uint32_t b = 1u << bit(j[k]), i = id[k] + (uint32_t)__popc(tw[k] & (b - 1u)) - base;
                    const uint32_t rank = r + (uint32_t)(k / U);
                    if (j[k] != kNone && (tw[k] & b) && i < nr) atomicOr(&s_row[i * MW + (rank >> 5)], 1u << (rank & 31u));
                }
            });
            __syncthreads();
            // neighbouring ranks of a row meet in a node of level h + 1, h their highest differing bit
            for (uint32_t i = tid; i < nr; i += NT) {
                uint32_t pred = kNone;
#pragma unroll 1
                for (uint32_t w = 0; w < MW; ++w)
                    for (uint32_t m = s_row[i * MW + w]; m; m &= m - 1u) {
                        const uint32_t r = w * 32u + (uint32_t)__builtin_ctz(m);
                        if (pred != kNone) {
                            const uint32_t h = 31u - (uint32_t)__clz(pred ^ r);
                            atomicAdd(&s_E[(lane & 15u) * EW + P - (P >> h) + (r >> (h + 1u))], 1u);
                        }
                        pred = r;
                    }
            }
            __syncthreads();
        }
        __syncthreads();
        for (uint32_t i = tid; i < W; i += NT) s_once[i] = s_twice[i] = 0u;
        pos = till;
        __syncthreads();
    }
    const uint32_t all = block_sum(ne, s_tot);
    if (tid == 0u && a.when != kWhenUnion) a.chunk_ne[chunk] = all;
    for (uint32_t i = tid; i + 1u < P; i += NT) {
        uint32_t n = 0u;
        for (uint32_t c = 0; c < 16u; ++c) n += s_E[c * EW + i];
        if (n) atomicAdd(&a.node_cnt[i], n);
    }
}

}  // namespace

// Tiles of equal width whose indices held twice are expected to fit the rows
// (of uniform streams; others may take rounds).
hipError_t acc_pairs_launch(AccArgs a, uint64_t sum_nnz, hipStream_t s)
{
    const uint32_t sl = a.P <= 16u ? 1u : a.P / 16u, mw = (16u * sl + 31u) / 32u;
    const double mu = (double)sum_nnz / (double)a.N, twice = 1.0 - (1.0 + mu) * std::exp(-mu);
    const uint64_t most = (uint64_t)std::min((double)kPairTile, std::max(4096.0, 0.75 * pair_rows(mw) / std::max(twice, 1e-6)));
    const uint64_t n = (a.chunk + most - 1u) / most;
    a.T = (uint32_t)std::min<uint64_t>(((a.chunk + n - 1u) / n + 1023u) & ~1023ull, kPairTile);
    const int slot = a.when == kWhenUnion ? kTReduceSlow : kTReducePass;
    timer_begin(slot, s);
    const auto k = sl == 1u ? k_pairs<1> : sl == 2u ? k_pairs<2> : sl == 4u ? k_pairs<4> : sl == 8u ? k_pairs<8> : k_pairs<16>;
    hipLaunchKernelGGL(k, dim3(a.nchunks), dim3(1024), 0, s, a);
    timer_end(slot, s);
    return hipGetLastError();
}

}  // namespace sparcml
