// Huffman stages of compression (FZModules Sec. 3.2: the Huffman encoder
// builds its code from the histogram of quantisation codes; FZMod-Default
// runs this on the CPU, here it runs on the GPU):
//   k_codebook - length-limited minimum-redundancy code lengths by
//                package-merge in one workgroup, canonical codewords;
//   k_encode   - chunked encoding (chunk = block) in one pass over the
//                codes, stream offsets by a look-back over tile groups,
//                words assembled in LDS;
//   k_finalize - tile-boundary words, outlier/patch sections, header, or
//                the verbatim container.
#include "fz_common.h"
#include "fz_kernels.h"

namespace fz {

// ------------------------------------------------------------ codebook
// Package-merge (Larmore & Hirschberg): leaves = used symbols sorted by
// (count, symbol); list[kLmax] = leaves; list[l] = merge(leaves,
// packages of list[l+1]) with equal weights putting the leaf first; select
// the first 2n-2 items of list[1], each selected package standing for the
// next two items one level deeper.  A symbol's length is the number of
// levels at which it is selected.  Leaves keep their sorted order in every
// list, so a level is summarised by the leaves' positions in it.
//
// One workgroup, bound by the latency of its serial steps and, at many used
// symbols, by the instructions its 16 waves issue, so the work follows the
// number of used symbols n: these are compacted first, and the sort runs
// over the next power of two.  A list is never stored: the lane that merges
// items 2i and 2i + 1 of list l adds them to package i of list l - 1, one
// barrier per level.  W is the type of the weights: a package weighs at
// most kLmax times the field's values, 32 bits up to 2^32 / kLmax values.
// Measured: 20 / 100 / 300 / 1000 used symbols 16.0 / 19.2 / 24.0 / 30.7 us
// with the launch, against 22.7 / 26 / 33 / 41 us with two full binary
// searches per level over stored lists (a step is about 250 cycles of LDS
// latency and dependent instructions, a level three barriers and reads on
// top) and LDS permutes in the sort.
struct PackageShared {
    uint16_t pos[kLmax][kBins + 2];  // [l]: position of leaf t in list l (1..kLmax-1); [kBins]: unused writes
    uint32_t take[kLmax + 1];
};

// Code length of leaf t (0 past the n leaves): thread t holds the weight of
// leaf t; leaf, p0 and p1 are LDS arrays of kBins.
template <class W>
__device__ uint32_t package_merge(W w, uint32_t n, W* leaf, W* p0, W* p1, PackageShared& sh) {
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const bool is_leaf = t < n;
    if (is_leaf) leaf[t] = w;
    __syncthreads();
    W* cur = p0;
    W* nxt = p1;
    uint32_t np = n / 2;
    if (t < np) cur[t] = leaf[2 * t] + leaf[2 * t + 1];
    __syncthreads();
    // leaves among the first 2 t items of the previous level's list.  Going
    // up a level a list only gains items, its packages only get lighter,
    // and this count only falls, by about half as much per level (1000
    // codes: at most 118, 49, 21, 9, 4, ... places), so the search starts
    // there and gallops down.
    // No branch inside the search: a step is the LDS latency and about ten
    // instructions, and every taken branch would add to it.
    constexpr uint32_t kHalve = 1u << 16;  // gallop step that halves the range
    const uint32_t d = 2 * t;
    uint32_t hint = n;
#pragma unroll 1
    for (int l = kLmax - 1; l >= 1; l--) {
        const uint32_t len = n + np;
        if (128 * wave < len) {
            uint32_t lo = d > np ? d - np : 0u, hi = min(hint, min(d, n)), g = hint == n ? kHalve : 1u;
            lo = d < len ? lo : hi;
            while (__ballot(lo < hi)) {
                // leaf m comes before package d - 1 - m
                const uint32_t m = hi - min(g, (hi - lo + 1) >> 1);
                const W a = leaf[min(m, (uint32_t)kBins - 1)], c = cur[min(d - 1 - m, (uint32_t)kBins - 1)];
                const bool before = a <= c, in = lo < hi;
                lo = in && before ? m + 1 : lo;
                hi = in && !before ? m : hi;
                g = before ? kHalve : min(2 * g, kHalve);
            }
            // the lane's items 2 t and 2 t + 1: leaf i or package j, the next
            const uint32_t i = lo, j = d - lo;
            hint = d < len ? i : n;
            const bool i0 = i < n, i1 = i + 1 < n, j0 = j < np, j1 = j + 1 < np;
            const W a0 = leaf[min(i, (uint32_t)kBins - 1)], a1 = leaf[min(i + 1, (uint32_t)kBins - 1)],
                    b0 = cur[min(j, (uint32_t)kBins - 1)], b1 = cur[min(j + 1, (uint32_t)kBins - 1)];
            const bool f0 = i0 & (!j0 | (a0 <= b0));                                   // the first is a leaf
            const bool f1 = f0 ? i1 & (!j0 | (a1 <= b0)) : i0 & (!j1 | (a0 <= b1));   // the second is
            sh.pos[l][f0 && d < len ? i : (uint32_t)kBins] = (uint16_t)d;
            sh.pos[l][f1 && d + 1 < len ? i + (f0 ? 1u : 0u) : (uint32_t)kBins] = (uint16_t)(d + 1);
            const W sum = (f0 ? a0 : b0) + (f1 ? (f0 ? a1 : a0) : (f0 ? b0 : b1));
            nxt[t] = sum;
        }
        __syncthreads();
        W* tmp = cur;
        cur = nxt;
        nxt = tmp;
        np = len / 2;
    }
    if (wave == 0) {
        // leaves among the first `take` items of each level, their positions
        // ascending: every step-th leaf, then those after the last of these
        const uint32_t step = (n + 63) / 64;
        uint32_t take = 2 * n - 2;
        uint32_t c[kLmax];
#pragma unroll
        for (int l = 1; l < kLmax; l++) c[l] = step * lane < n ? sh.pos[l][step * lane] : 0xFFFFu;
#pragma unroll
        for (int l = 1; l < kLmax; l++) {
            uint32_t k = (uint32_t)__popcll(__ballot(c[l] < take));
            if (step > 1 && k) {
                const uint32_t j = step * (k - 1) + lane;
                const uint32_t p = sh.pos[l][j < n ? j : 0];
                k = step * (k - 1) + (uint32_t)__popcll(__ballot(lane < step && j < n && p < take));
            }
            if (lane == 0) sh.take[l] = take;
            take = 2 * (take - k);
        }
        if (lane == 0) sh.take[kLmax] = take;
    }
    __syncthreads();
    uint32_t L = 0;
    if (is_leaf) {
#pragma unroll
        for (int l = 1; l < kLmax; l++) L += sh.pos[l][t] < sh.take[l] ? 1u : 0u;
        L += t < sh.take[kLmax] ? 1u : 0u;
    }
    return L;
}

// Bitonic stages inside a wave.  Both values of a pair are at hand in each of
// its lanes; `max_lanes` are the lanes that keep the larger one, and the
// comparison's ballot, flipped there, selects.
__device__ __forceinline__ uint64_t pick64(uint64_t lanes, uint64_t set, uint64_t clear) {
    return __builtin_amdgcn_inverse_ballot_w64(lanes) ? set : clear;
}
template <int J>
__device__ __forceinline__ uint64_t bitonic_stage(uint64_t v, uint64_t max_lanes) {
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    if (J >= 16) {
        // the swaps leave the pair's values in order in both lanes
        uint64_t a, b;
        if (J == 16) {
            const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
            a = (uint64_t)h[0] << 32 | l[0];
            b = (uint64_t)h[1] << 32 | l[1];
        } else {
            const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
            a = (uint64_t)h[0] << 32 | l[0];
            b = (uint64_t)h[1] << 32 | l[1];
        }
        return pick64(__ballot(b < a) ^ max_lanes, b, a);
    }
    // lane ^ 1, 2: quad permutes; ^ 4: mirror of 8 lanes, then of each quad;
    // ^ 8: rotation of the row of 16
    constexpr int kCtrl = J == 1 ? 0xB1 : (J == 2 ? 0x4E : (J == 4 ? 0x141 : 0x128));
    uint32_t ol = dpp32<kCtrl, 0xf>(lo), oh = dpp32<kCtrl, 0xf>(hi);
    if (J == 4) {
        ol = dpp32<0x1B, 0xf>(ol);
        oh = dpp32<0x1B, 0xf>(oh);
    }
    const uint64_t o = (uint64_t)oh << 32 | ol;
    return pick64(__ballot(o < v) ^ max_lanes, o, v);
}
// Lanes with bit J set.
template <int J>
constexpr uint64_t lanes_with() {
    uint64_t m = 0;
    for (int l = 0; l < 64; l++) m |= (uint64_t)((l & J) != 0) << l;
    return m;
}
// Stage J of the merge of size K < 64 (directions alternate inside the wave)
template <int K, int J>
__device__ __forceinline__ uint64_t stage_in(uint64_t v) {
    return bitonic_stage<J>(v, lanes_with<J>() ^ lanes_with<K>());
}
// The last six stages of a merge of 64 or more, `down`: descending.
__device__ __forceinline__ uint64_t merge_wave(uint64_t v, bool down) {
    const uint64_t f = down ? ~0ull : 0ull;
    v = bitonic_stage<32>(v, lanes_with<32>() ^ f);
    v = bitonic_stage<16>(v, lanes_with<16>() ^ f);
    v = bitonic_stage<8>(v, lanes_with<8>() ^ f);
    v = bitonic_stage<4>(v, lanes_with<4>() ^ f);
    v = bitonic_stage<2>(v, lanes_with<2>() ^ f);
    return bitonic_stage<1>(v, lanes_with<1>() ^ f);
}

__global__ __launch_bounds__(1024) void k_codebook(uint32_t* __restrict__ hist, uint8_t* __restrict__ out_lens,
                                                   uint32_t* __restrict__ cw, Misc* misc) {
    // the sort's two buffers, then (the sort done) the arrays of package_merge
    __shared__ uint64_t buf[3][kBins];
    __shared__ PackageShared ps;
    __shared__ uint8_t slen[kBins];
    __shared__ uint32_t s_first_unused, s_used[16];
    __shared__ uint64_t red[16];
    __shared__ CanonShared cs;

    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    auto add = [](uint64_t a, uint64_t b) { return a + b; };
    // sum the histogram copies; copy 0 keeps the total, the others are
    // cleared (at the end: a barrier waits for stores)
    uint32_t h = 0;
#pragma unroll
    for (int k = 0; k < kHistCopies; k++) h += hist[k * kBins + t];
    slen[t] = 0;
    if (t == 0) s_first_unused = kBins;
    const uint64_t um = __ballot(h > 0);
    const uint64_t wtotal = wave_incl_scan64(h, add);
    if (lane == 63) {
        s_used[wave] = (uint32_t)__popcll(um);
        red[wave] = wtotal;
    }
    __syncthreads();
    uint32_t n = 0, before = 0;
    uint64_t total = 0;
#pragma unroll
    for (uint32_t w = 0; w < 16; w++) {
        const uint32_t v = s_used[w];
        before += w < wave ? v : 0u;
        n += v;
        total += red[w];
    }

    if (n == 1) {
        if (h == 0) atomicMin(&s_first_unused, t);
        __syncthreads();
        if (h > 0) slen[t] = 1;
        if (t == s_first_unused) slen[t] = 1;
    } else if (n >= 2) {
        // the used symbols' keys (count << 10 | symbol), compacted, then a
        // bitonic sort over the next power of two (at least a wave), the
        // rest filled with the largest key; a thread keeps its key in a
        // register: partners closer than 64 are exchanged inside the wave,
        // farther ones through two alternating LDS buffers (one barrier per
        // such stage)
        const uint32_t P = n <= 64 ? 64u : 1u << (32 - __clz((int)(n - 1)));
        if (h > 0) buf[0][before + (uint32_t)__popcll(um & ((1ull << lane) - 1))] = ((uint64_t)h << 10) | t;
        __syncthreads();
        uint64_t v = t < n ? buf[0][t] : ~0ull;
        const bool part = 64 * wave < P;  // wave-uniform
        if (part) {
            v = stage_in<2, 1>(v);
            v = stage_in<4, 2>(v);
            v = stage_in<4, 1>(v);
            v = stage_in<8, 4>(v);
            v = stage_in<8, 2>(v);
            v = stage_in<8, 1>(v);
            v = stage_in<16, 8>(v);
            v = stage_in<16, 4>(v);
            v = stage_in<16, 2>(v);
            v = stage_in<16, 1>(v);
            v = stage_in<32, 16>(v);
            v = stage_in<32, 8>(v);
            v = stage_in<32, 4>(v);
            v = stage_in<32, 2>(v);
            v = stage_in<32, 1>(v);
            v = merge_wave(v, wave & 1);
        }
        int side = 1;
#pragma unroll 1
        for (uint32_t k = 128; k <= P; k <<= 1) {
            const bool down = (64 * wave & k) != 0;
#pragma unroll 1
            for (uint32_t j = k >> 1; j >= 64; j >>= 1) {
                uint64_t* kb = buf[side];
                if (part) kb[t] = v;
                __syncthreads();
                if (part) {
                    const uint64_t o = kb[t ^ j];
                    const bool keep_min = ((64 * wave & j) == 0) != down;
                    v = keep_min ? (o < v ? o : v) : (o > v ? o : v);
                }
                side ^= 1;
            }
            if (part) v = merge_wave(v, down);
        }
        __syncthreads();
        uint32_t L;
        if (total <= 0xFFFFFFFFull / kLmax)
            L = package_merge<uint32_t>(t < n ? (uint32_t)(v >> 10) : 0u, n, reinterpret_cast<uint32_t*>(buf[0]),
                                        reinterpret_cast<uint32_t*>(buf[1]), reinterpret_cast<uint32_t*>(buf[2]), ps);
        else
            L = package_merge<uint64_t>(t < n ? v >> 10 : 0ull, n, buf[0], buf[1], buf[2], ps);
        if (t < n) slen[v & 1023] = (uint8_t)L;
    }
    __syncthreads();
    const uint32_t len = slen[t];
    const uint32_t code = canonical_code(len, cs);
    cw[t] = code | (len << 16);
    // total stream bits = sum count * length
    const uint64_t bits = wave_incl_scan64((uint64_t)h * len, add);
    if (lane == 63) red[wave] = bits;
    if (t < 512) out_lens[t] = (uint8_t)(slen[2 * t] | (slen[2 * t + 1] << 4));
    __syncthreads();
    hist[t] = h;
#pragma unroll
    for (int k = 1; k < kHistCopies; k++) hist[k * kBins + t] = 0;
    if (t == 0) {
        uint64_t s = 0;
#pragma unroll
        for (int w = 0; w < 16; w++) s += red[w];
        misc->total_bits_cb = s;
    }
}

// --------------------------------------------------------------- encode
// words of one tile at most (every value at kLmax bits)
constexpr int kEncTileWords = kTileBlocks * kBlockElems * kLmax / 32;

// A lane's 8 codes of block b, segment s (from the start of the codes when
// the block or segment holds no values, so the load is unconditional and
// can be issued a tile ahead), and the number of real values among them.
template <int ND>
__device__ __forceinline__ uint4 load_codes(const uint16_t* __restrict__ codes, const Geom& g, uint32_t b,
                                            uint32_t s, uint32_t& nv) {
    nv = 0;
    if (b < g.nblocks) {
        BlockInfo info = block_info(g, b);
        seg_index<ND>(g, info, s, nv);
    }
    const uint64_t at = nv ? (uint64_t)b * kBlockElems + s * 8 : 0;
    return *reinterpret_cast<const uint4*>(&codes[at]);
}

// Single pass over the codes.  A workgroup takes T consecutive 4-block
// tiles: it reads their codes once (all loads issued together, kept packed
// in registers), writes the chunk table, publishes the group's bit count and
// obtains the group's stream offset by a decoupled look-back over groups,
// then writes the bits tile by tile.  A group publishes its count before it
// waits, and waits only on groups with lower workgroup index (dispatched
// before it), so the chain never waits on a workgroup that is not running;
// the wait is bounded anyway (F_TIMEOUT).
//
// A workgroup lives about 18 us, 63% of it waiting: for its codes, the
// look-back and the barriers between its phases.  The quantiser stores a
// code as the byte offset of its table entry (8 code), entries are a
// codeword and a length in two registers, codewords join in pairs of 32
// bits, and a lane's string is placed by three funnel shifts: 14 vector
// instructions per value instead of 24, which leaves large fields where they
// were (1024^3 0.79 ms, 512^3 0.15 ms) and helps small ones, whose workgroups
// run alone.  What did not help at 1024^3: 12 tiles per group (0.86 ms, the
// waves 105 instead of 89 registers), 6 (0.95), 5 waves per SIMD forced
// (0.89), look-back windows of 128 and 256 descriptors (0.95, 1.09); a window
// of 16 and longer sleeps: 0.86 -> 0.79 (every descriptor read goes to
// memory).  The bits are written in passes of up to kEncPass tiles; small
// fields take fewer tiles per group, see encode_tiles.
constexpr uint32_t kEncPass = 4;

// A lane's 8 codes of a segment with nv real values: the sum of their
// lengths; all: every lane's segment is full (uniform).
__device__ __forceinline__ uint2 code_entry(const uint2* CW, uint32_t off) {
    return *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(CW) + off);
}
__device__ __forceinline__ uint32_t code_bits(const uint4& pk, uint32_t nv, bool all, const uint2* CW) {
    const uint32_t o[8] = {pk.x & 0xFFFFu, pk.x >> 16, pk.y & 0xFFFFu, pk.y >> 16,
                           pk.z & 0xFFFFu, pk.z >> 16, pk.w & 0xFFFFu, pk.w >> 16};
    uint32_t l[8];
#pragma unroll
    for (int i = 0; i < 8; i++) l[i] = code_entry(CW, o[i]).y;
    if (!all) {
#pragma unroll
        for (int i = 0; i < 8; i++) l[i] = i < (int)nv ? l[i] : 0u;
    }
    return ((l[0] + l[1]) + (l[2] + l[3])) + ((l[4] + l[5]) + (l[6] + l[7]));
}

template <int ND, uint32_t T>
__global__ __launch_bounds__(256) void k_encode(const uint16_t* __restrict__ codes, Geom g,
                                                const uint32_t* __restrict__ cw_g, uint32_t ntiles, Misc* misc,
                                                uint8_t* __restrict__ out, uint64_t* desc,
                                                uint64_t* __restrict__ tile_start, uint32_t* __restrict__ tfirst,
                                                uint32_t* __restrict__ tlast) {
    constexpr uint32_t kPass = T < kEncPass ? T : kEncPass;
    static_assert(T % kPass == 0, "whole passes");
    constexpr int kWords = (int)kPass * kEncTileWords + 8;  // one pass (+ bit offset and window overrun)
    __shared__ uint2 CW[kBins];
    __shared__ uint32_t W[kWords];   // one pass of tiles
    __shared__ uint32_t s_carry[2];  // a pass's partial last word, for the next pass (by pass parity)
    __shared__ uint32_t wsum[T][4];
    __shared__ uint64_t s_excl;
    // an error bound the quantiser rejected: it wrote no codes, and what the
    // buffer holds are no table offsets (set before this kernel, so the same
    // for every workgroup)
    if (misc->flags & F_EB) return;
    uint16_t* chunks = reinterpret_cast<uint16_t*>(out + misc->off_chunks);
    uint32_t* stream = reinterpret_cast<uint32_t*>(out + misc->off_stream);
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t grp = blockIdx.x;
    const uint32_t tile0 = grp * T;
    // pass over the group's codes: every tile's codes loaded at once
    // (packed, 4 registers per tile, so the loads' latencies overlap), then
    // the tiles' bit counts and totals; the codeword entries are looked up
    // again when the bits are written
    uint4 pk[T];
    uint32_t partial = 0;             // tiles where some lane's segment is not full (uniform)
    uint32_t pre[(T + 1) / 2] = {};   // bits of the wave's earlier lanes, two tiles per register
#pragma unroll
    for (uint32_t k = 0; k < T; k++) {
        uint32_t nv;
        const uint32_t b = (tile0 + k) * kTileBlocks + wave;
        pk[k] = load_codes<ND>(codes, g, tile0 + k < ntiles ? b : g.nblocks, lane, nv);
        partial |= (__ballot(nv != 8) ? 1u : 0u) << k;
    }
    // real values of the lane's segment, again where they are not 8
    auto real_values = [&](uint32_t k) -> uint32_t {
        const uint32_t b = (tile0 + k) * kTileBlocks + wave;
        uint32_t nv = 0;
        if (tile0 + k < ntiles && b < g.nblocks) {
            const BlockInfo info = block_info(g, b);
            seg_index<ND>(g, info, lane, nv);
        }
        return nv;
    };
    for (uint32_t i = t; i < (uint32_t)kBins; i += 256) {
        const uint32_t e = cw_g[i];
        CW[i] = make_uint2(e & 0xFFFFu, e >> 16);
    }
    for (uint32_t i = t; i < (uint32_t)kWords; i += 256) W[i] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < T; k++) {
        const bool all = !((partial >> k) & 1u);
        const uint32_t nb = code_bits(pk[k], all ? 8u : real_values(k), all, CW);
        const uint32_t incl = wave_incl_scan(nb);
        pre[k / 2] |= (incl - nb) << (16 * (k & 1));  // at most 6144
        if (lane == 63) wsum[k][wave] = incl;
    }
    __syncthreads();
    // chunk table (block bit counts) from the tile totals: no store among
    // the phase's loads, whose waits would otherwise also cover it
    if (t < T * 4) {
        const uint32_t k = t >> 2, w = t & 3;
        const uint32_t b = (tile0 + k) * kTileBlocks + w;
        if (tile0 + k < ntiles && b < g.nblocks) chunks[b] = (uint16_t)wsum[k][w];
    }
    uint64_t gsum = 0;
    for (uint32_t k = 0; k < T; k++) gsum += wsum[k][0] + wsum[k][1] + wsum[k][2] + wsum[k][3];
    if (wave == 0) {
        const uint64_t ex = lookback<16, 8>(desc, grp, gsum, OpAdd(), &misc->flags);
        if (lane == 0) {
            s_excl = ex;
            if (tile0 + T >= ntiles) misc->total_bits_enc = ex + gsum;
        }
    }
    __syncthreads();
    // the bits, in passes of kPass tiles: each pass's tiles are OR-ed into
    // one LDS buffer (one barrier), then its words are stored as one
    // contiguous run.  The group's partial first and last words are shared
    // with the neighbouring groups and merged by k_finalize (tile_start of
    // the group's first tile; its other tiles start at 0, nothing to
    // merge); a pass's partial last word is carried into the next pass.
    const uint64_t G0 = s_excl;
    const uint32_t tend = min(tile0 + T, ntiles);  // past the group's last tile
    if (t < T && tile0 + t < ntiles) tile_start[tile0 + t] = t == 0 ? G0 : 0ull;
    uint64_t G = G0;
#pragma unroll
    for (uint32_t h = 0; h < T / kPass; h++) {
        const uint32_t k0 = h * kPass;
        if (tile0 + k0 >= ntiles) break;  // uniform
        const uint32_t shp = (uint32_t)(G & 31);
        uint32_t rel = 0;  // bits of the pass's earlier tiles
#pragma unroll
        for (uint32_t kk = 0; kk < kPass; kk++) {
            const uint32_t k = k0 + kk;
            const uint32_t tile = tile0 + k;
            if (tile >= ntiles) break;  // uniform
            uint32_t wpre = 0, bits = 0;
            for (uint32_t w = 0; w < 4; w++) {
                if (w < wave) wpre += wsum[k][w];
                bits += wsum[k][w];
            }
            if (t == 0 && tile != ntiles - 1 && bits < 32) atomicOr(&misc->flags, F_INTERNAL);
            // (keeps the first pass's eight offsets per tile from being held
            // in registers until here: 162 VGPRs, three waves per SIMD)
            asm volatile("" : "+v"(pk[k].x), "+v"(pk[k].y), "+v"(pk[k].z), "+v"(pk[k].w));
            const uint32_t o8[8] = {pk[k].x & 0xFFFFu, pk[k].x >> 16, pk[k].y & 0xFFFFu, pk[k].y >> 16,
                                    pk[k].z & 0xFFFFu, pk[k].z >> 16, pk[k].w & 0xFFFFu, pk[k].w >> 16};
            uint2 e8[8];
#pragma unroll
            for (int i = 0; i < 8; i++) e8[i] = code_entry(CW, o8[i]);
            uint32_t nv = 8;
            if ((partial >> k) & 1u) {  // uniform
                nv = real_values(k);
#pragma unroll
                for (int i = 0; i < 8; i++)
                    if (i >= (int)nv) e8[i] = make_uint2(0, 0);
            }
            if (nv) {
                // pairs (at most 24 bits), then the lane's two strings of 4
                // codewords (at most 48 bits)
                uint32_t pr[4], pl[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    pr[i] = e8[2 * i].x << e8[2 * i + 1].y | e8[2 * i + 1].x;
                    pl[i] = e8[2 * i].y + e8[2 * i + 1].y;
                }
                const uint64_t a0 = (uint64_t)pr[0] << pl[1] | pr[1], a1 = (uint64_t)pr[2] << pl[3] | pr[3];
                const uint32_t n0 = pl[0] + pl[1], n1 = pl[2] + pl[3];  // n0 >= 1; a1 = 0 when n1 = 0
                // left-aligned in three words, then shifted right by the bit
                // offset o into words w0 .. w0 + 3 (o + n0 + n1 <= 127)
                const uint64_t b1 = a1 << ((64 - n1) & 63);
                const uint64_t s01 = a0 << (64 - n0) | b1 >> n0;
                const uint32_t s2 = (uint32_t)((b1 << (64 - n0)) >> 32);
                const uint32_t s0 = (uint32_t)(s01 >> 32), s1 = (uint32_t)s01;
                const uint32_t p = shp + rel + wpre + ((pre[k / 2] >> (16 * (k & 1))) & 0xFFFFu);  // from the pass's first word
                const uint32_t o = p & 31, w0 = p >> 5;
                const uint32_t o0 = s0 >> o, o1 = __builtin_amdgcn_alignbit(s0, s1, o),
                               o2 = __builtin_amdgcn_alignbit(s1, s2, o), o3 = __builtin_amdgcn_alignbit(s2, 0, o);
                atomicOr(&W[w0], o0);
                if (o1) atomicOr(&W[w0 + 1], o1);
                if (o2) atomicOr(&W[w0 + 2], o2);
                if (o3) atomicOr(&W[w0 + 3], o3);
            }
            rel += bits;
        }
        __syncthreads();
        // the pass's words: the first one shares bits with the previous
        // pass (carried) or group (parked in tfirst), the last one with the
        // next pass (carried) or group (parked in tlast of the group's last
        // tile); the field's very last word is stored
        const bool last_pass = tile0 + k0 + kPass >= tend;
        const uint32_t nwords = (shp + rel + 31) >> 5;
        const bool end_part = ((shp + rel) & 31) != 0;
        const uint64_t wbase = G >> 5;
        // pass h reads the slot pass h - 1 wrote and writes the other one:
        // the writer of this pass's carry may run before every thread has
        // read the previous one
        const uint32_t carry_in = s_carry[(h + 1) & 1];
        for (uint32_t w = t; w < nwords; w += 256) {
            uint32_t v = W[w];
            W[w] = 0;
            const bool first = w == 0 && shp != 0, last = w == nwords - 1 && end_part;
            if (first && h > 0) v |= carry_in;
            if (first && h == 0) tfirst[tile0] = v;
            else if (last && !last_pass) s_carry[h & 1] = v;
            else if (last && tend != ntiles) tlast[tend - 1] = v;
            else stream[wbase + w] = v;
        }
        G += rel;
        __syncthreads();
    }
}

// -------------------------------------------------------------- verbatim
// The verbatim container: header (flag bit 0) and the raw floats, written by
// the whole finalize grid.
__device__ void write_verbatim(const Geom& g, uint32_t mode, double eb, uint32_t pred, uint32_t hflags,
                               const Misc* misc, const float* __restrict__ x, uint8_t* __restrict__ out, int vec,
                               uint64_t gid, uint64_t stride) {
    if (gid == 0) {
        double eb_abs;
        resolve_eb(mode, eb, misc->mm_lo, misc->mm_hi, &eb_abs);
        uint8_t h[kHdr];
        for (int k = 0; k < kHdr; k++) h[k] = 0;
        auto st32 = [&](int o, uint32_t v) { for (int k = 0; k < 4; k++) h[o + k] = (uint8_t)(v >> (8 * k)); };
        auto st64 = [&](int o, uint64_t v) { for (int k = 0; k < 8; k++) h[o + k] = (uint8_t)(v >> (8 * k)); };
        st32(0, kMagic);
        h[4] = (uint8_t)kVersion;
        h[5] = (uint8_t)(kVersion >> 8);
        h[6] = (uint8_t)hflags;
        st32(8, g.ndim);
        st32(12, pred);
        st64(16, g.n[0]);
        st64(24, g.n[1]);
        st64(32, g.n[2]);
        st32(40, mode);
        st32(44, kRadius);
        st64(48, __double_as_longlong(eb));
        st64(56, __double_as_longlong(eb_abs));
        st64(64, (uint64_t)kHdr + 4 * g.N);
        uint4* dst = reinterpret_cast<uint4*>(out);
        const uint4* src = reinterpret_cast<const uint4*>(h);
        for (int k = 0; k < kHdr / 16; k++) dst[k] = src[k];
    }
    float* o = reinterpret_cast<float*>(out + kHdr);
    if (vec) {
        const f32x4* x4 = reinterpret_cast<const f32x4*>(x);
        f32x4* o4 = reinterpret_cast<f32x4*>(o);
        for (uint64_t i = gid; i < g.N / 4; i += stride) o4[i] = x4[i];
        for (uint64_t i = (g.N & ~3ull) + gid; i < g.N; i += stride) o[i] = x[i];
    } else {
        for (uint64_t i = gid; i < g.N; i += stride) o[i] = x[i];
    }
}

// ------------------------------------------------------------- finalize
// Layout from the device-side counts; boundary words shared by two tiles;
// outlier and patch sections compacted from the per-tile staging slots in
// tile order (= position order); zero padding; header.  When the packed
// container would not be smaller than the raw floats only the verbatim
// decision is recorded for the host.
__global__ __launch_bounds__(256) void k_finalize(Geom g, uint32_t mode, double eb, uint32_t pred, Misc* misc,
                                                  uint8_t* out, uint32_t ntiles, const uint64_t* __restrict__ tile_start,
                                                  const uint32_t* __restrict__ tfirst,
                                                  const uint32_t* __restrict__ tlast,
                                                  const uint32_t* __restrict__ tile_cnt,
                                                  const uint64_t* __restrict__ tile_off,
                                                  const uint2* __restrict__ ostage, const uint2* __restrict__ pstage,
                                                  const uint8_t* __restrict__ bpred,
                                                  const uint64_t* __restrict__ reg_idx,
                                                  const int32_t* __restrict__ coef, const float* __restrict__ x,
                                                  int xvec, uint32_t codec) {
    const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t flags = misc->flags;
    const bool shuffle = codec != 0;
    // Huffman: stream bits; bit-shuffle: kept words (no bit count)
    const uint64_t bits = shuffle ? 0 : misc->total_bits_enc;
    const uint64_t words = shuffle ? misc->total_bits_enc : (bits + 31) / 32;
    const uint64_t nout = misc->n_out, npat = misc->n_pat, nreg = misc->nreg;
    // a per-block choice of first-order Lorenzo everywhere is written as a
    // first-order container (no map)
    if (pred_has_map(pred) && misc->map_off) pred = 0;
    const bool has_map = pred_has_map(pred);
    const Layout L = shuffle ? make_speed_layout(g.nblocks, words, nout, npat)
                             : make_layout(g.nblocks, has_map, nreg, words, nout, npat);
    const bool verbatim = (flags & F_OVERFLOW) || L.total >= (uint64_t)kHdr + 4 * g.N;
    if (gid == 0) {
        if (!shuffle && (bits != misc->total_bits_cb || L.chunks != misc->off_chunks))
            atomicOr(&misc->flags, F_INTERNAL);
        misc->verbatim = verbatim ? 1 : 0;
        misc->total_bytes = verbatim ? (uint64_t)kHdr + 4 * g.N : L.total;
    }
    if (flags & (F_NONFINITE | F_EB | F_INTERNAL | F_TIMEOUT)) return;
    if (verbatim) {
        write_verbatim(g, mode, eb, pred, shuffle ? 1u | kFlagShuffle : 1u, misc, x, out, xvec, gid, stride);
        return;
    }

    // predictor map (2 bits per block) and regression coefficients
    if (has_map)
        for (uint64_t i = gid; i < ((uint64_t)g.nblocks + 3) / 4; i += stride) {
            uint8_t v = 0;
            for (int k = 0; k < 4; k++) {
                const uint64_t b = 4 * i + k;
                if (b < g.nblocks) v |= (uint8_t)((bpred[b] & 3) << (2 * k));
            }
            out[L.map + i] = v;
        }
    if (nreg)
        for (uint64_t b = gid; b < g.nblocks; b += stride) {
            const bool reg = pred == 2 || (has_map && bpred[b] == 2);
            if (!reg) continue;
            const uint64_t r = pred == 2 ? b : reg_idx[b];
            reinterpret_cast<int4*>(out + L.coef)[r] = reinterpret_cast<const int4*>(coef)[b];
        }
    uint32_t* stream = reinterpret_cast<uint32_t*>(out + L.stream);
    for (uint64_t i = gid + 1; !shuffle && i < ntiles; i += stride) {
        const uint64_t G = tile_start[i];
        if (G & 31) stream[G >> 5] = tlast[i - 1] | tfirst[i];
    }
    uint32_t* o_pos = reinterpret_cast<uint32_t*>(out + L.opos);
    int32_t* o_val = reinterpret_cast<int32_t*>(out + L.oval);
    uint32_t* p_pos = reinterpret_cast<uint32_t*>(out + L.ppos);
    uint32_t* p_bits = reinterpret_cast<uint32_t*>(out + L.pbits);
    if (nout | npat) {
        const uint32_t lane = threadIdx.x & 63;
        const uint64_t wid = gid >> 6, nw = stride >> 6;
        const uint64_t m31 = (1ull << 31) - 1;
        for (uint64_t tile = wid; tile < ntiles; tile += nw) {
            const uint32_t c = tile_cnt[tile];
            if (!c) continue;
            const uint64_t off = tile_off[tile];
            const uint64_t slot = tile * (uint64_t)(kTileBlocks * kBlockElems);
            const uint32_t co = c & 0xFFFFu, cp = c >> 16;
            // four entries per lane and pass, all loads issued before the
            // stores (the copy is latency-bound otherwise)
            for (uint32_t j0 = 0; j0 < co; j0 += 256) {
                uint2 a[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t j = j0 + lane + 64 * k;
                    a[k] = j < co ? ostage[slot + j] : make_uint2(0, 0);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t j = j0 + lane + 64 * k;
                    if (j < co) {
                        o_pos[(off & m31) + j] = a[k].x;
                        o_val[(off & m31) + j] = (int32_t)a[k].y;
                    }
                }
            }
            for (uint32_t j0 = 0; j0 < cp; j0 += 256) {
                uint2 a[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t j = j0 + lane + 64 * k;
                    a[k] = j < cp ? pstage[slot + j] : make_uint2(0, 0);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t j = j0 + lane + 64 * k;
                    if (j < cp) {
                        p_pos[(off >> 31) + j] = a[k].x;
                        p_bits[(off >> 31) + j] = a[k].y;
                    }
                }
            }
        }
    }
    if (gid == 0) {
        // zero padding between and after sections
        const uint64_t ends[8] = {L.map + (has_map ? ((uint64_t)g.nblocks + 3) / 4 : 0), L.coef + 16 * nreg,
                                  L.chunks + (shuffle ? 4 * kMaskWords : 2) * (uint64_t)g.nblocks,
                                  L.stream + 4 * words, L.opos + 4 * nout, L.oval + 4 * nout, L.ppos + 4 * npat,
                                  L.pbits + 4 * npat};
        const uint64_t starts[8] = {L.coef, L.chunks, L.stream, L.opos, L.oval, L.ppos, L.pbits, L.total};
        for (int k = shuffle ? 2 : 0; k < 8; k++)
            for (uint64_t a = ends[k]; a < starts[k]; a++) out[a] = 0;
        // header
        double eb_abs;
        resolve_eb(mode, eb, misc->mm_lo, misc->mm_hi, &eb_abs);
        uint8_t h[kHdr];
        for (int k = 0; k < kHdr; k++) h[k] = 0;
        auto st32 = [&](int o, uint32_t v) { for (int k = 0; k < 4; k++) h[o + k] = (uint8_t)(v >> (8 * k)); };
        auto st64 = [&](int o, uint64_t v) { for (int k = 0; k < 8; k++) h[o + k] = (uint8_t)(v >> (8 * k)); };
        st32(0, kMagic);
        h[4] = (uint8_t)kVersion;
        h[5] = (uint8_t)(kVersion >> 8);
        h[6] = shuffle ? (uint8_t)kFlagShuffle : 0;
        st32(8, g.ndim);
        st32(12, pred);
        st64(16, g.n[0]);
        st64(24, g.n[1]);
        st64(32, g.n[2]);
        st32(40, mode);
        st32(44, kRadius);
        st64(48, __double_as_longlong(eb));
        st64(56, __double_as_longlong(eb_abs));
        st64(64, L.total);
        st32(72, g.nblocks);
        st32(76, (uint32_t)nout);
        st32(80, (uint32_t)npat);
        st32(84, (uint32_t)words);
        st64(88, bits);
        st32(96, (uint32_t)nreg);
        uint4* dst = reinterpret_cast<uint4*>(out);
        const uint4* src = reinterpret_cast<const uint4*>(h);
        for (int k = 0; k < kHdr / 16; k++) dst[k] = src[k];
    }
}

// ------------------------------------------------------------ launchers
void launch_codebook(hipStream_t st, uint32_t* hist, uint8_t* out_lens, uint32_t* cw, Misc* misc) {
    hipLaunchKernelGGL(k_codebook, dim3(1), dim3(1024), 0, st, hist, out_lens, cw, misc);
}

void launch_encode(hipStream_t st, int grid, const uint16_t* codes, const Geom& g, const uint32_t* cw, Misc* misc,
                   uint32_t ntiles, uint8_t* out, uint64_t* desc, uint64_t* tile_start, uint32_t* tfirst,
                   uint32_t* tlast) {
    (void)grid;  // one workgroup per group of tiles
    const uint32_t groups = encode_groups(ntiles), T = encode_tiles(ntiles);
#define FZ_ENC(NDV, TV)                                                                                             \
    hipLaunchKernelGGL((k_encode<NDV, TV>), dim3(groups), dim3(256), 0, st, codes, g, cw, ntiles, misc, out, desc, \
                       tile_start, tfirst, tlast)
#define FZ_ENC_T(NDV)            \
    if (T == 8) FZ_ENC(NDV, 8); \
    else if (T == 4) FZ_ENC(NDV, 4); \
    else FZ_ENC(NDV, 1)
    if (g.ndim == 3) {
        FZ_ENC_T(3);
    } else if (g.ndim == 2) {
        FZ_ENC_T(2);
    } else {
        FZ_ENC_T(1);
    }
#undef FZ_ENC_T
#undef FZ_ENC
}

uint32_t encode_groups(uint32_t ntiles) {
    const uint32_t T = encode_tiles(ntiles);
    return (ntiles + T - 1) / T;
}

void launch_finalize(hipStream_t st, const Geom& g, uint32_t mode, double eb, uint32_t pred, Misc* misc,
                     uint8_t* out, uint32_t ntiles, const uint64_t* tile_start, const uint32_t* tfirst,
                     const uint32_t* tlast, const uint32_t* tile_cnt, const uint64_t* tile_off, const uint2* ostage,
                     const uint2* pstage, const uint8_t* bpred, const uint64_t* reg_idx, const int32_t* coef,
                     const float* x, uint32_t codec) {
    // about four tiles per wave for the outlier/patch compaction
    uint32_t grid = (ntiles + 15) / 16;
    if (grid < 1024) grid = 1024;
    if (grid > 8192) grid = 8192;
    hipLaunchKernelGGL(k_finalize, dim3(grid), dim3(256), 0, st, g, mode, eb, pred, misc, out, ntiles, tile_start,
                       tfirst, tlast, tile_cnt, tile_off, ostage, pstage, bpred, reg_idx, coef, x,
                       (int)(((uintptr_t)x & 15) == 0), codec);
}

}  // namespace fz
