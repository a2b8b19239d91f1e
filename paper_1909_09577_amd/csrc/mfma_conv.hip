// Matrix-core implicit-GEMM engine for the forward pass and the input gradient.
//
// Both passes are the same contraction
//     out[b, m, t] = sum_r sum_k  W'[m, r, k] * in[b, r, t*stride - padL + k*dil]
// with (m, r) = (co, ci), W' = w, padL = pad for the forward pass and, for the input gradient
// of a stride-1 convolution, (m, r) = (ci, co), W'[ci,co,k] = w[co,ci,K-1-k],
// padL = dil*(K-1) - pad, in = dz (materialised by the caller of this engine).
//
// Work decomposition (one workgroup = 4 wavefronts of 64 lanes, one workgroup per CU, one
// wavefront per SIMD with up to 512 registers, persistent over work items):
//   * an output tile is 64 channels x NT*32 time steps of one batch item, accumulated by one
//     wavefront in 2*NT 32x32 MFMA accumulators;
//   * work items: every wavefront first computes some tiles on its own over all reduction chunks
//     (no exchange with the others: the unrolled kernels only), then the four wavefronts of a
//     workgroup share tiles by splitting the reduction channels in chunks of 32 (wave w takes chunks
//     w, w+4, ...), sum the four partial tiles through LDS at the end of the tile and finish a
//     quarter of the rows each; neither form has a workgroup barrier in its main loop;
//   * the activation window of a chunk (32 channels x all time steps the K taps touch) is read
//     once with 16-byte buffer loads along T (lanes outside the row are sent out of range and read
//     zeros) and written to the wavefront's private LDS region transposed to [time][channel], so
//     that every tap is a row offset and each MFMA B fragment (8 consecutive channels of one time
//     step) is one aligned 16-byte LDS read; the next chunk (of this work item or the next one) is
//     staged while the current one is multiplied;
//   * weights are prepacked once per call into MFMA A-fragment order and stream from L2 straight
//     into registers (each lane reads 16 contiguous bytes, a wavefront 1 KiB); a fragment register
//     set is reloaded right after its last use with the data of its next use, across chunks and
//     work items;
//   * tiles are numbered channel-tile fastest, so the workgroups that the hardware places on one
//     XCD (blockIdx mod 8) keep reusing the same slice of the packed weights in that L2.
// Two forms of the main loop: for the tap counts of the Jasper blocks (KT > 0) a chunk is one
// straight-line block of 4*NT*KT MFMAs with every load, LDS write and wait placed between them;
// for any other K (KT == 0) tap pairs run in a loop with staging in out-of-line blocks.
#include "../../include/nm_conv1d.h"
#include "conv_tile.h"

#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <utility>

namespace nm {
namespace {

struct TileCoords {
    int mt, b, t0, ws_al, off0;
};

// KT > 0: the number of taps is a compile-time constant and a chunk is one straight-line block
// (see the unrolled main loop below); KT == 0: any K, tap pairs in a loop.
// LEN: the instance for ragged calls (per-sample lengths); of the unrolled kernels it
// alone carries the test for tiles in the padding.
// STATS: the instance that also writes the per-tile statistics of its stored outputs (ConvGemmParams::stats).
// ANYROW: rows of any length (the test for output rows of that kind costs the other calls of few tiles about 1 %;
// conv_split_kernel and the K=1 kernel's instance for lengths make it at run time).
// PADPAIR: of the tap-pair kernels' ANYROW instances, the one where a wavefront may have an odd number of tap pairs (see do_pair).
template <int NT, int STRIDE, int KT, bool LEN = false, bool STATS = false, bool ANYROW = false, bool PADPAIR = false>
__global__ __launch_bounds__(kThreads) void conv_gemm_kernel(const ConvGemmParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int TN = NT * 32;

    const int nitems = p.nitems;                           // staging items per lane and chunk
    const int nmy = (p.nch - wave + kWaves - 1) / kWaves;  // chunks of this wavefront (may be 0)
    const int P = p.Kp >> 1;                               // tap pairs per chunk
    const int tap_bytes = p.dil * kRowBytes;
    const int gstep = (int)(gridDim.x % (unsigned)p.nmt);  // tile += gridDim.x moves the channel tile by this much
    const __amdgpu_buffer_rsrc_t rs_in =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)((size_t)p.B * p.R * p.Tin * 2), 0x00020000);

    // staging item `it` of a lane: channel pair pp = lane & 15, time group q0 + 4*it (8 steps)
    auto buf_ptr = [&](int par) { return smem + ((size_t)(par & 1) * kWaves + wave) * p.buf_bytes; };

    auto finish_coords = [&](TileCoords &tc, int tt) {
        tc.t0 = tt * TN;
        const int ws = tc.t0 * STRIDE - p.padL;
        tc.ws_al = (ws >> 3) * 8;  // arithmetic shift: floor
        tc.off0 = ws - tc.ws_al;
    };
    auto tile_coords = [&](int tile, int &tt) {
        TileCoords tc;
        tc.mt = tile % p.nmt;
        const int ntile = tile / p.nmt;
        tc.b = ntile / p.ntt;
        tt = ntile - tc.b * p.ntt;
        finish_coords(tc, tt);
        return tc;
    };
    // Staging loads of chunk c of batch item b, window start ws_al.  The scalar part of the address
    // (batch item, chunk) travels as the scalar offset of the buffer load; lanes whose 8 time steps
    // or whose channel lie outside the tensor get an offset beyond the buffer and read zeros.
    struct StageAddr {
        uint32_t soff, va, vb;  // scalar offset; lane offsets of the even / odd channel (or out of range)
        int tq;                 // first time step of item 0 of this lane
        int tlen;               // valid length of the batch item (Tin without lengths)
        int ws_al;              // time step of window row 0
    };
    auto stage_addr = [&](int b, int c, int ws_al) {
        StageAddr a;
        a.soff = (uint32_t)(((size_t)b * p.R + (size_t)c * kChunk) * p.Tin * 2);
        const int rem = p.R - c * kChunk;  // channels left from this chunk on
        const int l = fresh_lane();
        const int pp = l & 15, q0 = l >> 4;
        const uint32_t base = (uint32_t)(((2 * pp) * p.Tin + 8 * q0 + ws_al) * 2);
        const int tq = ws_al + 8 * q0;
        a.va = 2 * pp < rem ? base : kOutOfRange;
        a.vb = 2 * pp + 1 < rem ? base + (uint32_t)(p.Tin * 2) : kOutOfRange;
        a.tq = tq;
        a.tlen = __builtin_amdgcn_readfirstlane(clipped_len(p.len_in, b, p.Tin));
        a.ws_al = ws_al;
        return a;
    };
    auto stage_load = [&](const StageAddr &a, int it, bool active, u32x4 &xa, u32x4 &xb) {
        const int t = a.tq + 32 * it;
        // a group is requested when it starts inside [0, tlen) (groups are 8-aligned and Tin % 8 == 0, so it
        // then ends inside the row); what lies at or beyond tlen in it is cleared when it is written to LDS
        const bool t_ok = active && (unsigned)t < (unsigned)a.tlen;
        // a lane of a missing channel holds kOutOfRange: adding 64*it keeps it beyond the buffer
        xa = __builtin_amdgcn_raw_buffer_load_b128(rs_in, t_ok ? a.va + (uint32_t)(64 * it) : kOutOfRange, a.soff, 0);
        xb = __builtin_amdgcn_raw_buffer_load_b128(rs_in, t_ok ? a.vb + (uint32_t)(64 * it) : kOutOfRange, a.soff, 0);
    };
    // transposing write of an item: one dword (channel pair) per time step
    auto stage_write = [&](unsigned char *buf, int it, bool active, const u32x4 &xa, const u32x4 &xb) {
        const int l = fresh_lane();
        const int pp = l & 15, q0 = l >> 4;
        const uint32_t row = active ? (uint32_t)(q0 * 8 + it * 32) : (uint32_t)(nitems * 32);  // idle writes go to the dump rows
        uint32_t *dst = reinterpret_cast<uint32_t *>(buf + row * kRowBytes + pp * 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            dst[(2 * j) * kRowDwords] = zip_lo16(xa[j], xb[j]);
            dst[(2 * j + 1) * kRowDwords] = zip_hi16(xa[j], xb[j]);
        }
    };
    // the same with the lane's LDS offsets computed by the caller: lane_lds = ((lane/16)*8 rows,
    // channel pair lane%16) for real items, lane_dump = (first dump row, channel pair) for idle ones
    auto stage_write_at = [&](unsigned char *buf, uint32_t lane_lds, uint32_t lane_dump, int it, bool active,
                              const u32x4 &xa, const u32x4 &xb) {
        uint32_t *dst = reinterpret_cast<uint32_t *>(buf + (active ? lane_lds + (uint32_t)(it * 32 * kRowBytes) : lane_dump));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            dst[(2 * j) * kRowDwords] = zip_lo16(xa[j], xb[j]);
            dst[(2 * j + 1) * kRowDwords] = zip_hi16(xa[j], xb[j]);
        }
    };
    // With lengths, the 8-step group that contains the first padding sample has been staged whole: its
    // rows from the valid length on are cleared here, after the chunk's items are in LDS and before it
    // is read (groups that start in the padding were never requested).  ws_al: time of buffer row 0.
    auto clear_padding_rows = [&](unsigned char *buf, int tlen, int ws_al) {
        const int r0 = tlen - ws_al;                 // first padding row of the window
        const int nr = ((tlen + 7) & ~7) - tlen;     // rows up to the end of its group (0 when tlen % 8 == 0)
        if (tlen < p.Tin && nr > 0 && r0 >= 0 && r0 < nitems * 32) {
            const int l = fresh_lane();
            for (int r = l >> 4; r < nr; r += 4)
                *reinterpret_cast<uint32_t *>(buf + (size_t)(r0 + r) * kRowBytes + (l & 15) * 4) = 0u;
        }
    };
    constexpr int kSlots = KT > 0 ? unrolled_slots(KT) : 6;  // staging items of the next chunk held in registers
    u32x4 sxa[kSlots], sxb[kSlots];
    // a whole chunk, nothing to overlap with (first tile, or every tile without cross-tile staging)
    auto stage_chunk_now = [&](int b, int c, int ws_al, unsigned char *buf) {
        const StageAddr sa = stage_addr(b, c, ws_al);
        for (int it0 = 0; it0 < nitems; it0 += kSlots) {
#pragma unroll
            for (int q = 0; q < kSlots; ++q) stage_load(sa, it0 + q, it0 + q < nitems, sxa[q], sxb[q]);
#pragma unroll
            for (int q = 0; q < kSlots; ++q) stage_write(buf, it0 + q, it0 + q < nitems, sxa[q], sxb[q]);
        }
        clear_padding_rows(buf, sa.tlen, sa.ws_al);
    };

    // ---- weight fragment stream: buffer loads whose scalar offset is a cursor into the packed weights
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (int)p.wp_bytes, 0x00020000);
    const uint32_t w_lane = (uint32_t)lane * 16;
    auto w_load = [&](uint32_t soff, int f) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_lane + (uint32_t)f * 1024u, soff, 0));
    };

    // (KT == 0)  Tap pairs are multiplied alternately from two register sets
    // (afA, afB: [tap 2][ks 2][mi 2] fragments each); a set is reloaded right after its last use
    // with the pair that comes two pairs later in this wavefront's stream, which runs across
    // chunks and tiles, so the loads have about two pairs of MFMA work to arrive.  A tile with an
    // odd number of pairs gets one pair of zero weights, so that tiles start on afA.  The cursor
    // is kept in scalar registers and moves without branches except at a tile end; the loads are
    // buffer loads whose scalar offset is the cursor.
    bf16x8 afA[8], afB[8];
    const int total_pairs = nmy * P;
    const int slots = total_pairs + (total_pairs & 1);  // pairs per tile including the zero pair
    constexpr uint32_t kPairBytes = 512 * 16;           // one tap pair of one chunk
    const uint32_t zero_soff = (uint32_t)(p.wp_zero * 16);
    const uint32_t chunk_jump = kPairBytes * (uint32_t)(1 + (kWaves - 1) * P);  // last pair of a chunk -> first of the next
    auto w_base = [&](int mt) { return (uint32_t)(mt * p.nch + wave) * (uint32_t)P * kPairBytes; };
    int w_tile = blockIdx.x, w_mt = (int)(blockIdx.x % (unsigned)p.nmt), w_pr = 0, w_s = 0;
    bool w_live = w_tile < p.num_tiles && nmy > 0;
    uint32_t w_soff = w_base(w_mt);
    auto w_next = [&]() -> uint32_t {  // offset of the cursor pair; moves the cursor on
        const uint32_t off = (w_live && w_s < total_pairs) ? w_soff : zero_soff;
        ++w_s;
        ++w_pr;
        const bool chunk_end = w_pr == P;
        w_soff += chunk_end ? chunk_jump : kPairBytes;
        w_pr = chunk_end ? 0 : w_pr;
        if (__builtin_expect(w_s == slots, 0)) {  // tile end
            w_s = 0;
            w_pr = 0;
            w_tile += gridDim.x;
            w_mt += gstep;
            w_mt -= w_mt >= p.nmt ? p.nmt : 0;
            w_live = w_live && w_tile < p.num_tiles;
            w_soff = w_base(w_mt);
        }
        return off;
    };
    if constexpr (KT == 0) {
        const uint32_t s0 = w_next();
#pragma unroll
        for (int f = 0; f < 8; ++f) afA[f] = w_load(s0, f);
        const uint32_t s1 = w_next();
#pragma unroll
        for (int f = 0; f < 8; ++f) afB[f] = w_load(s1, f);
    }


    // (KT > 0)  One register set of four fragments ([ks 2][mi 2]) per tap, rotating over NS sets
    // plus one extra set for each of the KT % NS last taps, so that the assignment of taps to sets
    // is the same in every chunk.  A set is reloaded right after its last multiplication with the
    // tap that uses it next: NS taps later in this chunk, or in the next chunk of this wavefront's
    // stream (w_cur / w_nxt: byte offsets of the current and the next chunk), which runs across
    // tiles.  The zero tap that pads an odd K in the packed tensor is never touched.
    constexpr int NS = 4, NQ = KT / NS, NR = KT % NS, NSETS = KT > 0 ? NS + NR : 1;
    bf16x8 wf[NSETS][4];
    constexpr uint32_t kTapBytes = 4 * 64 * 16;
    const uint32_t chunk_bytes = (uint32_t)p.Kp * kTapBytes;
    auto chunk_off = [&](int mt, int c) { return (uint32_t)(mt * p.nch + c) * chunk_bytes; };
    uint32_t w_cur = 0;

    Epilogue<NT> epi;
    epi.init(p.out, p.res, p.scale, p.shift, p.B, p.M, p.Tout, p.relu, p.len_out, p.len_out_div, p.stats);

    int cc = 0;  // chunks this wavefront has consumed so far: chunk number cc uses buffer cc & 1
    // accumulators: zero here, and again in the epilogue as soon as a tile's values have been handed over
    f32x16 acc[2][NT];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

    // ---- work items of this wavefront.  First `full` private tiles: tile k*4G + wave*G + blockIdx
    // (G workgroups), computed by this wavefront alone over every reduction chunk, so they need no
    // exchange between wavefronts; then the shared tiles 4G*full + blockIdx + j*G, whose reduction
    // chunks the four wavefronts split (chunk wave, wave+4, ...) and whose partial sums they add
    // through LDS.  With 1280 tiles on 256 CUs that is one private tile per wavefront and one
    // shared tile per workgroup: four fifths of the work skip the exchange.  Both numberings keep
    // tile mod (channel tiles) = blockIdx mod (channel tiles) when G is a multiple of it, i.e.
    // one slice of the packed weights per XCD.
    const int G = (int)gridDim.x;
    const int nA = KT > 0 ? p.full : 0;
    const int tilesA = nA * kWaves * G;
    auto item_tile = [&](int k) {
        return k < nA ? (k * kWaves + wave) * G + (int)blockIdx.x : tilesA + (int)blockIdx.x + (k - nA) * G;
    };
    auto first_chunk = [&](bool priv) { return priv ? 0 : wave; };
    int item = 0, tile = item_tile(0);
    int tt_unused = 0;
    TileCoords tc_next = tile_coords(tile < p.num_tiles ? tile : 0, tt_unused);
    if (tile < p.num_tiles && p.overlap && (nA > 0 || nmy > 0))
        stage_chunk_now(tc_next.b, first_chunk(nA > 0), tc_next.ws_al, buf_ptr(0));
    if constexpr (KT > 0) {
        if (tile < p.num_tiles && (nA > 0 || nmy > 0)) {
            w_cur = chunk_off(tc_next.mt, first_chunk(nA > 0));
#pragma unroll
            for (int k = 0; k < NS; ++k)
#pragma unroll
                for (int f = 0; f < 4; ++f) wf[k][f] = w_load(w_cur + (uint32_t)k * kTapBytes, f);
#pragma unroll
            for (int e = 0; e < NR; ++e)
#pragma unroll
                for (int f = 0; f < 4; ++f) wf[NS + e][f] = w_load(w_cur + (uint32_t)(NS * NQ + e) * kTapBytes, f);
        }
    }

    for (; tile < p.num_tiles; ++item) {
        const bool priv = item < nA;
        const bool next_priv = item + 1 < nA;
        const int next_tile = item_tile(item + 1);
        const TileCoords tc = tc_next;
        const bool next_ok = p.overlap && next_tile < p.num_tiles;
        tc_next = tile_coords(next_tile < p.num_tiles ? next_tile : tile, tt_unused);
        const TileCoords tn = tc_next;
        tile = next_tile;

        if (!p.overlap && nmy > 0) stage_chunk_now(tc.b, wave, tc.ws_al, buf_ptr(cc));

        if constexpr (KT > 0) {
            // A tile that lies wholly in the padding of its batch item -- every input sample its window covers is at or
            // beyond the valid length (forward), or every output position is at or beyond the output limit (input
            // gradient) -- needs no arithmetic: its accumulators stay zero (the staged window is zero) or its outputs are
            // written as zeros.  It still runs ONE chunk, which keeps the pipeline (staging of the next item's first
            // chunk, weight sets) exactly as it is for a live tile.
            bool dead = false;
            if constexpr (LEN) {
                if (p.len_in) dead = tc.t0 * STRIDE - p.padL >= clipped_len(p.len_in, tc.b, p.Tin);
                if (p.len_out) dead = dead || tc.t0 >= epi.out_limit(tc.b);
            }
            const int n_full = priv ? p.nch : nmy;  // chunks of this item for this wavefront
            const int n_ch = dead ? min(n_full, 1) : n_full;
            auto chunk_of = [&](int i) { return priv ? i : wave + kWaves * i; };
            if (n_ch > 0) {
                // ---- unrolled main loop: one chunk (KT taps, 4*NT*KT MFMAs) is a single straight-line
                // block, so staging loads, staging writes, weight reloads and LDS reads are placed
                // between the MFMAs by the compiler and every wait counts exactly what is in flight.
                // The six staging items of the next chunk are requested one per tap during the
                // first six taps and written one per tap during the last six.
                static_assert(KT == 0 || KT >= 11, "the staging schedule needs eleven taps");
                const int ll = fresh_lane();
                const int lane_off = ((ll & 31) * STRIDE + tc.off0) * kRowBytes + (ll >> 5) * 16;
                const uint32_t lane_lds = (uint32_t)(((ll >> 4) * 8) * kRowBytes + (ll & 15) * 4);
                const uint32_t lane_dump = (uint32_t)(nitems * 32 * kRowBytes + (ll & 15) * 4);
                for (int ci = 0; ci < n_ch; ++ci) {
                    const bool more = ci + 1 < n_ch;
                    const bool has_t = more || next_ok;  // is there a chunk to stage for
                    const int c_nxt = more ? chunk_of(ci + 1) : first_chunk(next_priv);
                    const uint32_t w_nxt = has_t ? chunk_off(more ? tc.mt : tn.mt, c_nxt) : w_cur;
                    StageAddr sa = stage_addr(more ? tc.b : tn.b, c_nxt, more ? tc.ws_al : tn.ws_al);
                    sa.va = has_t ? sa.va : kOutOfRange;
                    sa.vb = has_t ? sa.vb : kOutOfRange;
                    const unsigned char *bbase = buf_ptr(cc) + lane_off;
                    unsigned char *nxt = buf_ptr(cc + 1);
                    bf16x8 b0[NT], b1[NT];
                    auto read_b = [&](bf16x8(&dst)[NT], int k, int ks) {
                        const unsigned char *brow = bbase + (size_t)k * tap_bytes + ks * 32;
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni)
                            dst[ni] = *reinterpret_cast<const bf16x8 *>(brow + ni * 32 * STRIDE * kRowBytes);
                    };
                    auto mma = [&](const bf16x8 &a0, const bf16x8 &a1, const bf16x8(&bf)[NT]) {
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni)
                            acc[0][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, bf[ni], acc[0][ni], 0, 0, 0);
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni)
                            acc[1][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, bf[ni], acc[1][ni], 0, 0, 0);
                    };
                    wave_lds_fence();  // the staged chunk is visible to every lane
                    read_b(b0, 0, 0);
                    auto tap = [&](auto kc) {
                        constexpr int k = decltype(kc)::value;
                        constexpr int set = k < NS * NQ ? k % NS : NS + (k - NS * NQ);
                        // the tap that uses this set next
                        constexpr bool same_chunk = k < NS * NQ && k + NS < NS * NQ;
                        constexpr int next_tap = same_chunk ? k + NS : (k < NS * NQ ? k % NS : k);
                        const uint32_t src = (same_chunk ? w_cur : w_nxt) + (uint32_t)next_tap * kTapBytes;
                        // (a scheduling barrier per k-step keeps every load where it is written: the
                        // compiler would otherwise move the reloads down to their use)
                        read_b(b1, k, 1);
                        mma(wf[set][0], wf[set][1], b0);
                        wf[set][0] = w_load(src, 0);
                        wf[set][1] = w_load(src, 1);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (k + 1 < KT) read_b(b0, k + 1, 0);
                        mma(wf[set][2], wf[set][3], b1);
                        wf[set][2] = w_load(src, 2);
                        wf[set][3] = w_load(src, 3);
                        if constexpr (k < kSlots) stage_load(sa, k, k < nitems, sxa[k], sxb[k]);
                        if constexpr (k >= KT - kSlots) {
                            constexpr int it = k - (KT - kSlots);
                            stage_write_at(nxt, lane_lds, lane_dump, it, has_t && it < nitems, sxa[it], sxb[it]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    for_each_index(tap, std::make_integer_sequence<int, (KT > 0 ? KT : 1)>{});
                    if (has_t) clear_padding_rows(nxt, sa.tlen, sa.ws_al);
                    w_cur = w_nxt;
                    ++cc;
                }
            }
        } else if (nmy > 0) {
            // ---- main loop over (chunk, tap pair): 4 k-steps of 16 channels = 8*NT MFMAs per pair
            // (the packed weights pad an odd K with one zero tap).  All MFMAs sit in this loop.
            const int ll = fresh_lane();
            const int lane_off = ((ll & 31) * STRIDE + tc.off0) * kRowBytes + (ll >> 5) * 16;
            int ci_ord = 0, pr = 0;
            // where the staging items of this chunk go: the next chunk of this tile, or the first
            // chunk of the next tile, or nowhere
            bool has_t = nmy > 1 || next_ok;
            const bool async_stage = P > kSlots / 2;  // shorter chunks stage the next one at their end
            int t_b = nmy > 1 ? tc.b : tn.b, t_ws = nmy > 1 ? tc.ws_al : tn.ws_al, t_c = nmy > 1 ? wave + kWaves : wave;
            const unsigned char *bbase = buf_ptr(cc) + lane_off;
            unsigned char *nxt = buf_ptr(cc + 1);
            bf16x8 b0[NT], b1[NT];
            auto read_b = [&](bf16x8(&dst)[NT], int k, int ks) {
                const unsigned char *brow = bbase + (size_t)k * tap_bytes + ks * 32;
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
                    dst[ni] = *reinterpret_cast<const bf16x8 *>(brow + ni * 32 * STRIDE * kRowBytes);
            };
            auto mma = [&](const bf16x8 &a0, const bf16x8 &a1, const bf16x8(&bf)[NT]) {
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) acc[0][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, bf[ni], acc[0][ni], 0, 0, 0);
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) acc[1][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, bf[ni], acc[1][ni], 0, 0, 0);
            };
            // one tap pair from the register set `af`; `real` is false only for the zero pad pair
            auto do_pair = [&](bf16x8(&af)[8], bool real) {
                // Staging of the next chunk: its items are requested at the first pair of this chunk
                // (static register slots) and written to LDS two at a time at the top of the last
                // three pairs, so the loads have most of a chunk (several microseconds) to arrive.
                // The writes come first in program order and only in pairs after the first, which
                // lets the wait they need leave the latest weight loads in flight.
                if (__builtin_expect(has_t && async_stage && pr >= P - kSlots / 2, 0)) {
#pragma unroll
                    for (int gq = 0; gq < kSlots / 2; ++gq) {
                        if (pr == P - kSlots / 2 + gq) {
#pragma unroll
                            for (int e = 0; e < 2; ++e)
                                if (2 * gq + e < nitems) stage_write(nxt, 2 * gq + e, true, sxa[2 * gq + e], sxb[2 * gq + e]);
                        }
                    }
                }
                if (__builtin_expect(pr == 0 && has_t && async_stage, 0)) {
                    const StageAddr sa = stage_addr(t_b, t_c, t_ws);
#pragma unroll
                    for (int it = 0; it < kSlots; ++it)
                        if (it < nitems) stage_load(sa, it, true, sxa[it], sxb[it]);
                }
                const int k = 2 * pr;
                // The second tap of an odd filter's last pair, and the pad pair: zeros times samples, a NaN where the sample
                // is infinite.  The ANYROW instances, whose calls ran on kernels without such products before, take the
                // last tap's samples (which the output is made of anyway), resp. zeros (in an
                // instance of its own: clearing costs 2 of the 52 us of 32 x 256 -> 256 channels, K=7, T=801).
                const int k1 = ANYROW ? min(k + 1, p.K - 1) : k + 1;
                auto keep = [&](bf16x8(&bf)[NT]) {
                    if constexpr (PADPAIR) {
                        const uint32_t mask = real ? ~0u : 0u;
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni) bf[ni] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, bf[ni]) & mask);
                    }
                };
                read_b(b1, k, 1);
                keep(b0);
                mma(af[0], af[1], b0);
                const uint32_t wn = w_next();
                af[0] = w_load(wn, 0);
                af[1] = w_load(wn, 1);
                read_b(b0, k1, 0);
                keep(b1);
                mma(af[2], af[3], b1);
                af[2] = w_load(wn, 2);
                af[3] = w_load(wn, 3);
                read_b(b1, k1, 1);
                keep(b0);
                mma(af[4], af[5], b0);
                af[4] = w_load(wn, 4);
                af[5] = w_load(wn, 5);
                read_b(b0, min(k + 2, p.Kp - 1), 0);
                keep(b1);
                mma(af[6], af[7], b1);
                af[6] = w_load(wn, 6);
                af[7] = w_load(wn, 7);
                if (__builtin_expect(real && ++pr == P, 0)) {  // end of a chunk
                    if (has_t) {
                        // windows longer than the register slots, or everything when chunks are short
                        for (int it = async_stage ? kSlots : 0; it < nitems; ++it) {
                            u32x4 ya, yb;
                            const StageAddr sl = stage_addr(t_b, t_c, t_ws);
                            stage_load(sl, it, true, ya, yb);
                            stage_write(nxt, it, true, ya, yb);
                        }
                        clear_padding_rows(nxt, clipped_len(p.len_in, t_b, p.Tin), t_ws);
                    }
                    ++ci_ord;
                    ++cc;
                    pr = 0;
                    has_t = false;
                    if (ci_ord < nmy) {
                        const bool more = ci_ord + 1 < nmy;
                        has_t = more || next_ok;
                        t_b = more ? tc.b : tn.b;
                        t_ws = more ? tc.ws_al : tn.ws_al;
                        t_c = more ? wave + kWaves * (ci_ord + 1) : wave;
                        bbase = buf_ptr(cc) + lane_off;
                        nxt = buf_ptr(cc + 1);
                        wave_lds_fence();
                        read_b(b0, 0, 0);
                    }
                }
            };
            wave_lds_fence();
            read_b(b0, 0, 0);
            for (int g = 0; g < total_pairs; g += 2) {
                do_pair(afA, true);
                do_pair(afB, g + 1 < total_pairs);
            }
        }

        // ---- epilogue (see Epilogue above).  The LDS tile lies in a staging buffer that holds no
        // live data: when the next item's first chunk has been staged into parity cc & 1, the other one.
        const int el = fresh_lane();  // nothing lane-dependent is kept alive across the main loop for this
        const int dead_par = next_ok ? ((cc & 1) ^ 1) : 0;
        float *tp = reinterpret_cast<float *>(smem + ((size_t)dead_par * kWaves + wave) * p.buf_bytes);

        if (priv) {
            // A private tile: this wavefront holds all 64 rows.
            epi.template store_private_tile<STATS, ANYROW>(acc, tp, el, tc.b, tc.t0, tc.mt * kTileM, tc.b * p.ntt + tc.t0 / TN);
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
        } else {
            // A shared tile.  Wave g finishes accumulator rows [4g, 4g+4) of every 32x32 block: each
            // wave hands the other three quarters over through LDS, one row of blocks (mi) per
            // round; the scratch is the dead-parity staging buffers of all four wavefronts.  The
            // operands of this wave's 16 rows are requested before the sum.
            const auto ld = epi.template request_rows<ANYROW>(el, tc.b, tc.t0, tc.mt * kTileM + 8 * wave, true);
            f32x4 *red = reinterpret_cast<f32x4 *>(smem + (size_t)dead_par * kWaves * p.buf_bytes);
            __syncthreads();  // every wavefront has left the main loop
            // One copy of the exchange per wave number, so that the accumulator quarters are named
            // statically and nothing has to be merged between the copies.
            auto exchange = [&](auto wave_const) {
                constexpr int Gw = decltype(wave_const)::value;
                f32x4 own[2][NT];
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
                    for (int g = 0; g < kWaves; ++g) {
                        if (g != Gw) {
                            const int slot = Gw < g ? Gw : Gw - 1;  // position of this wave among the three senders of quarter g
#pragma unroll
                            for (int ni = 0; ni < NT; ++ni) {
                                f32x4 v = {acc[mi][ni][4 * g], acc[mi][ni][4 * g + 1], acc[mi][ni][4 * g + 2],
                                           acc[mi][ni][4 * g + 3]};
                                red[((g * 3 + slot) * NT + ni) * 64 + el] = v;
                            }
                        }
                    }
                    __syncthreads();
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni)
                        own[mi][ni] = f32x4{acc[mi][ni][4 * Gw], acc[mi][ni][4 * Gw + 1], acc[mi][ni][4 * Gw + 2],
                                            acc[mi][ni][4 * Gw + 3]};
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni)  // this row of blocks is done: ready for the next tile
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
#pragma unroll
                    for (int slot = 0; slot < 3; ++slot) {
#pragma unroll
                        for (int ni = 0; ni < NT; ++ni) own[mi][ni] += red[((Gw * 3 + slot) * NT + ni) * 64 + el];
                    }
                    __syncthreads();  // scratch is reused by the next round / the transpose tile / the next tile's staging
                }
                epi.put_quarter(tp, el, own);
            };
            switch (wave) {
            case 0: exchange(std::integral_constant<int, 0>{}); break;
            case 1: exchange(std::integral_constant<int, 1>{}); break;
            case 2: exchange(std::integral_constant<int, 2>{}); break;
            default: exchange(std::integral_constant<int, 3>{}); break;
            }
            wave_lds_fence();
            epi.template finish_rows<STATS, ANYROW>(el, tp, ld);
            wave_lds_fence();
            if constexpr (STATS) {  // this wavefront's rows: channels 8*wave .. +7 of both row blocks of the tile
                epi.emit_row_stats(el, tp, tc.mt * kTileM + 8 * wave + (el >> 3) * 32 + (el & 7), tc.b * p.ntt + tc.t0 / TN,
                                   tc.t0);
                wave_lds_fence();
            }
        }
    }
}

// ---- calls whose tiles do not fill the chip ------------------------------------------------------
// conv_gemm_kernel gives a workgroup one tile of 160 time steps at a time, four chunks of reduction channels side by
// side: one utterance (600 steps, 768 channels) is 48 tiles on 256 CUs, and a layer with 64 input channels
// keeps two of its four wavefronts busy.  Here the reduction channels are also split over `nsplit` workgroups, the
// four wavefronts of a workgroup share ONE staged window and split the taps and halves of a chunk between them
// (wavefront w: channel half w & 1 of the taps w >> 1, (w >> 1) + 2, ...), so that a chunk of 32 channels is enough
// work for a workgroup; two workgroups fit a CU and cover each other's waits.  Tiles are 64 channels x NT*32
// steps, NT chosen for little padding.  The wavefronts add their sums through LDS as in conv_gemm_kernel; with
// nsplit > 1 the sums go to the workspace and split_reduce_kernel adds the parts in a fixed order and finishes (a few
// columns of tiles at a time where the workspace has no room for all of them: a tile's sums are the same either way).
// Workgroups that read the same weights sit on one XCD (blockIdx % 8) where the counts divide.
constexpr int kSplitRows = 256;   // staged rows of a window at most
constexpr int kSplitItems = kSplitRows / 8 * 16 / kThreads;  // staging items (8 steps x 2 channels) per lane and chunk

template <int NT, int STRIDE>
__global__ __launch_bounds__(kThreads, 2) void conv_split_kernel(const ConvGemmParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int TN = NT * 32;
    const int ncombo = p.nmt * p.nsplit, ncols = p.ncols;
    int combo, col;
    if (ncombo % 8 == 0) {
        const int j = (int)blockIdx.x >> 3;
        col = j % ncols;
        combo = (j / ncols) * 8 + ((int)blockIdx.x & 7);
    } else {
        combo = (int)blockIdx.x % ncombo;
        col = (int)blockIdx.x / ncombo;
    }
    const int mt = combo / p.nsplit, split = combo - mt * p.nsplit;
    const int b = (p.col0 + col) / p.ntt, t0 = (p.col0 + col - b * p.ntt) * TN;
    const int c0 = (int)((long)split * p.nch / p.nsplit), c1 = (int)((long)(split + 1) * p.nch / p.nsplit);

    Epilogue<NT> epi;
    epi.init(p.out, p.res, p.scale, p.shift, p.B, p.M, p.Tout, p.relu, p.len_out, p.len_out_div);
    const __amdgpu_buffer_rsrc_t rs_in =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)((size_t)p.B * p.R * p.Tin * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (int)p.wp_bytes, 0x00020000);

    const int ws = t0 * STRIDE - p.padL;
    const int ws_al = (ws >> 3) * 8;
    const int tlen = __builtin_amdgcn_readfirstlane(clipped_len(p.len_in, b, p.Tin));
    const int ngroups = p.nitems;  // 8-row groups of the window

    u32x4 sxa[kSplitItems], sxb[kSplitItems];
    auto stage_load = [&](int c) {
        const uint32_t soff = (uint32_t)(((size_t)b * p.R + (size_t)c * kChunk) * p.Tin * 2);
        const int rem = p.R - c * kChunk;
#pragma unroll
        for (int q = 0; q < kSplitItems; ++q) {
            const int idx = (int)threadIdx.x + kThreads * q;
            const int pp = idx & 15, grp = idx >> 4;
            const int t = ws_al + 8 * grp;
            const bool ok = grp < ngroups && (unsigned)t < (unsigned)tlen;
            const uint32_t at = (uint32_t)(((2 * pp) * p.Tin + t) * 2);
            sxa[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, ok && 2 * pp < rem ? at : kOutOfRange, soff, 0);
            sxb[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, ok && 2 * pp + 1 < rem ? at + (uint32_t)(p.Tin * 2) : kOutOfRange, soff, 0);
        }
    };
    auto stage_write = [&](unsigned char *buf) {
#pragma unroll
        for (int q = 0; q < kSplitItems; ++q) {
            const int idx = (int)threadIdx.x + kThreads * q;
            const int pp = idx & 15, grp = idx >> 4;
            if (grp >= ngroups) continue;
            const int nv = tlen - (ws_al + 8 * grp);  // valid steps of the group (a group before the row holds zeros)
            uint32_t *dst = reinterpret_cast<uint32_t *>(buf + (size_t)(8 * grp) * kRowBytes + pp * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t keep = nv >= 2 * j + 2 ? 0xffffffffu : (nv == 2 * j + 1 ? 0x0000ffffu : 0u);
                const uint32_t a = sxa[q][j] & keep, c = sxb[q][j] & keep;
                dst[(2 * j) * kRowDwords] = zip_lo16(a, c);
                dst[(2 * j + 1) * kRowDwords] = zip_hi16(a, c);
            }
        }
    };

    // this wavefront's units of a chunk: j -> tap (wave>>1) + 2j, channel half wave & 1; four register sets of two
    // fragments in rotation, each reloaded right after its use with the unit that uses it next, across chunks
    const int nu = (p.K + 1 - (wave >> 1)) >> 1;
    constexpr uint32_t kUnitStep = 4 * 2 * 1024;
    const uint32_t chunk_bytes = (uint32_t)p.Kp * 4096u;
    const uint32_t w_lane = (uint32_t)lane * 16 + (uint32_t)wave * 2048u;
    auto chunk_off = [&](int c) { return (uint32_t)(mt * p.nch + c) * chunk_bytes; };
    bf16x8 wf[4][2];
    auto w_load = [&](uint32_t soff, int mi) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_lane + (uint32_t)mi * 1024u, soff, 0));
    };
    f32x16 acc[2][NT];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

    // a tile that lies wholly in the padding of its batch item: its sums are zero
    bool dead = p.len_in && ws >= tlen;
    dead = dead || (p.len_out && t0 >= epi.out_limit(b));
    if (!dead) {
        stage_load(c0);
        uint32_t w_cur = chunk_off(c0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) wf[j][mi] = w_load(w_cur + (uint32_t)(j < nu ? j : 0) * kUnitStep, mi);  // (K = 1: the zero tap)
        stage_write(smem);
        __syncthreads();
        const uint32_t tap_step = 2u * (uint32_t)p.dil * kRowBytes;
        const uint32_t lane_off = (uint32_t)(((lane & 31) * STRIDE + ws - ws_al + (wave >> 1) * p.dil) * kRowBytes +
                                             (lane >> 5) * 16 + (wave & 1) * 32);
        for (int c = c0; c < c1; ++c) {
            const bool more = c + 1 < c1;
            const uint32_t w_nxt = more ? chunk_off(c + 1) : w_cur;
            const unsigned char *bbase = smem + (size_t)((c - c0) & 1) * p.buf_bytes + lane_off;
            if (more) stage_load(c + 1);
            bf16x8 bf[2][NT];
            auto read_b = [&](bf16x8(&dst)[NT], int j) {
                const unsigned char *at = bbase + (uint32_t)j * tap_step;
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) dst[ni] = *reinterpret_cast<const bf16x8 *>(at + ni * 32 * STRIDE * kRowBytes);
            };
            auto step = [&](auto set_c, int j) {
                constexpr int set = decltype(set_c)::value;
                read_b(bf[(set & 1) ^ 1], j + 1 < nu ? j + 1 : j);
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][mi], bf[set & 1][ni], acc[mi][ni], 0, 0, 0);
                const uint32_t src = j + 4 < nu ? w_cur + (uint32_t)(j + 4) * kUnitStep : w_nxt + (uint32_t)set * kUnitStep;
                wf[set][0] = w_load(src, 0);
                wf[set][1] = w_load(src, 1);
                __builtin_amdgcn_sched_barrier(0);
            };
            if (nu > 0) read_b(bf[0], 0);
            for (int j = 0; j < nu; j += 4) {
                step(std::integral_constant<int, 0>{}, j);
                if (j + 1 >= nu) break;
                step(std::integral_constant<int, 1>{}, j + 1);
                if (j + 2 >= nu) break;
                step(std::integral_constant<int, 2>{}, j + 2);
                if (j + 3 >= nu) break;
                step(std::integral_constant<int, 3>{}, j + 3);
            }
            if (more) stage_write(smem + (size_t)((c + 1 - c0) & 1) * p.buf_bytes);
            w_cur = w_nxt;
            __syncthreads();
        }
    }

    // sum over the wavefronts: wavefront g finishes accumulator rows 4g .. 4g+3 of every block, one row of blocks a round
    f32x4 *red = reinterpret_cast<f32x4 *>(smem);
    f32x4 own[2][NT];
    auto exchange = [&](auto wave_const) {
        constexpr int Gw = decltype(wave_const)::value;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
            for (int g = 0; g < kWaves; ++g) {
                if (g == Gw) continue;
                const int slot = Gw < g ? Gw : Gw - 1;
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
                    red[((g * 3 + slot) * NT + ni) * 64 + lane] =
                        f32x4{acc[mi][ni][4 * g], acc[mi][ni][4 * g + 1], acc[mi][ni][4 * g + 2], acc[mi][ni][4 * g + 3]};
            }
            __syncthreads();
#pragma unroll
            for (int ni = 0; ni < NT; ++ni)
                own[mi][ni] = f32x4{acc[mi][ni][4 * Gw], acc[mi][ni][4 * Gw + 1], acc[mi][ni][4 * Gw + 2], acc[mi][ni][4 * Gw + 3]};
#pragma unroll
            for (int slot = 0; slot < 3; ++slot)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) own[mi][ni] += red[((Gw * 3 + slot) * NT + ni) * 64 + lane];
            __syncthreads();
        }
    };
    switch (wave) {
    case 0: exchange(std::integral_constant<int, 0>{}); break;
    case 1: exchange(std::integral_constant<int, 1>{}); break;
    case 2: exchange(std::integral_constant<int, 2>{}); break;
    default: exchange(std::integral_constant<int, 3>{}); break;
    }
    if (p.nsplit > 1) {
        f32x4 *dst = p.part + ((((size_t)split * ncols + col) * p.nmt + mt) * kWaves + wave) * (2 * NT) * 64 + lane;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) dst[(mi * NT + ni) * 64] = own[mi][ni];
        return;
    }
    const auto ld = epi.template request_rows<true>(lane, b, t0, mt * kTileM + 8 * wave, true);
    float *tp = reinterpret_cast<float *>(smem) + wave * 16 * TN;
    epi.put_quarter(tp, lane, own);
    wave_lds_fence();
    epi.template finish_rows<false, true>(lane, tp, ld);
}

// ---- the strided first layer, enough tiles ----------------------------------------------------------------
// The encoder's first layer (64 channels, stride 2, K = 11) has 22 MFMA steps per chunk and two chunks, its input gradient (both
// parities at once, six taps) 12 and eight: in conv_split_kernel a workgroup spends more time waiting for its first window, adding its wavefronts' sums and finishing than multiplying.  Here
// the wavefronts of a workgroup share the staged window too, but each has rows (WM of them 64 rows each) and columns (4/WM of them
// 64 steps each) of its own, over all taps and channels: nothing is exchanged, and a window is staged once for 64*WM rows.
// Windows are double buffered, one barrier per chunk; weights come in fragment order from L2, six register sets in rotation, all
// steps of a chunk in a straight line (in a loop over the taps a step took 45 ns an MFMA instead of 20).  Columns of 96 and 128 steps
// were slower everywhere: two workgroups share a CU and cover each other's waits.  64 -> 256 channels, K=11, B=32, T=1600:
// forward 26.2 -> 16.3 us, the gradient's contraction 21.5 -> 17.3.
template <int STRIDE, int WM, int KT>
struct RowsShape {
    static constexpr int NT = 2, TN = NT * 32, WC = kWaves / WM, COLS = WC * TN;
    static constexpr int GROUPS = ((COLS - 1) * STRIDE + KT + 7 + 7) / 8;      // 8-row groups of a window
    static constexpr int kItems = (GROUPS * 16 + kThreads - 1) / kThreads;      // staging items per lane and chunk
    static constexpr int BUF = GROUPS * 8 * kRowBytes, TILE = kWaves * 16 * TN * 4;
    static constexpr int LDS = 2 * BUF > TILE ? 2 * BUF : TILE;
};

template <int STRIDE, int WM, int KT>
__global__ __launch_bounds__(kThreads, 2) void conv_rows_kernel(const ConvGemmParams p)
{
    using Sh = RowsShape<STRIDE, WM, KT>;
    constexpr int NT = Sh::NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wc = wave / WM;
    const int nmg = (p.nmt + WM - 1) / WM;
    const int col = (int)blockIdx.x / nmg, mt = ((int)blockIdx.x - col * nmg) * WM + wm;
    const int b = col / p.ntt, tw = (col - b * p.ntt) * Sh::COLS, t0 = tw + wc * Sh::TN;  // of the workgroup, of the wavefront

    Epilogue<NT> epi;
    epi.init(p.out, p.res, p.scale, p.shift, p.B, p.M, p.Tout, p.relu, p.len_out, p.len_out_div);
    const __amdgpu_buffer_rsrc_t rs_in =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)((size_t)p.B * p.R * p.Tin * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (int)p.wp_bytes, 0x00020000);
    const int ws = tw * STRIDE - p.padL, ws_al = (ws >> 3) * 8;
    const int tlen = __builtin_amdgcn_readfirstlane(clipped_len(p.len_in, b, p.Tin));

    u32x4 sxa[Sh::kItems], sxb[Sh::kItems];
    auto stage_load = [&](int c) {
        const uint32_t soff = (uint32_t)(((size_t)b * p.R + (size_t)c * kChunk) * p.Tin * 2);
        const int rem = p.R - c * kChunk;
#pragma unroll
        for (int q = 0; q < Sh::kItems; ++q) {
            const int idx = (int)threadIdx.x + kThreads * q;
            const int pp = idx & 15, grp = idx >> 4;
            const int t = ws_al + 8 * grp;
            const bool ok = grp < Sh::GROUPS && (unsigned)t < (unsigned)tlen;
            const uint32_t at = (uint32_t)(((2 * pp) * p.Tin + t) * 2);
            sxa[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, ok && 2 * pp < rem ? at : kOutOfRange, soff, 0);
            sxb[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, ok && 2 * pp + 1 < rem ? at + (uint32_t)(p.Tin * 2) : kOutOfRange, soff, 0);
        }
    };
    auto stage_write = [&](unsigned char *buf) {
#pragma unroll
        for (int q = 0; q < Sh::kItems; ++q) {
            const int idx = (int)threadIdx.x + kThreads * q;
            const int pp = idx & 15, grp = idx >> 4;
            if (kThreads * (q + 1) > Sh::GROUPS * 16 && grp >= Sh::GROUPS) continue;
            const int nv = tlen - (ws_al + 8 * grp);  // valid steps of the group (a group before the row holds zeros)
            uint32_t *dst = reinterpret_cast<uint32_t *>(buf + (size_t)(8 * grp) * kRowBytes + pp * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t keep = nv >= 2 * j + 2 ? 0xffffffffu : (nv == 2 * j + 1 ? 0x0000ffffu : 0u);
                const uint32_t a = sxa[q][j] & keep, c = sxb[q][j] & keep;
                dst[(2 * j) * kRowDwords] = zip_lo16(a, c);
                dst[(2 * j + 1) * kRowDwords] = zip_hi16(a, c);
            }
        }
    };

    // steps of a chunk: step j is tap j / 2, channel half j % 2
    constexpr int steps = 2 * KT;
    constexpr uint32_t kStep = 2048;
    const uint32_t chunk_bytes = (uint32_t)p.Kp * 4096u;
    auto chunk_off = [&](int c) { return (uint32_t)(min(mt, p.nmt - 1) * p.nch + c) * chunk_bytes; };
    constexpr int NS = 6;  // register sets
    bf16x8 wf[NS][2];
    auto w_load = [&](uint32_t soff, int mi) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, (uint32_t)lane * 16 + (uint32_t)mi * 1024u, soff, 0));
    };
    f32x16 acc[2][NT];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

    // (uniform over the workgroup: a window that lies wholly in the padding, or columns that are zero whatever the sums)
    const bool dead = (p.len_in && ws >= tlen) || (p.len_out && tw >= epi.out_limit(b));
    if (!dead) {
        stage_load(0);
        uint32_t w_cur = chunk_off(0);
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) wf[j][mi] = w_load(w_cur + (uint32_t)j * kStep, mi);
        stage_write(smem);
        __syncthreads();
        const uint32_t lane_off = (uint32_t)((((lane & 31) + wc * Sh::TN) * STRIDE + ws - ws_al) * kRowBytes + (lane >> 5) * 16);
        for (int c = 0; c < p.nch; ++c) {
            const bool more = c + 1 < p.nch;
            const uint32_t w_nxt = more ? chunk_off(c + 1) : w_cur;
            const unsigned char *bbase = smem + (c & 1) * Sh::BUF + lane_off;
            if (more) stage_load(c + 1);
            bf16x8 bf[2][NT];
            auto read_b = [&](bf16x8(&dst)[NT], int j) {
                const unsigned char *at = bbase + (j >> 1) * kRowBytes + (j & 1) * 32;
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) dst[ni] = *reinterpret_cast<const bf16x8 *>(at + ni * 32 * STRIDE * kRowBytes);
            };
            read_b(bf[0], 0);
            for_each_index([&](auto index) __attribute__((always_inline)) {
                constexpr int j = decltype(index)::value, set = j % NS;
                if constexpr (j + 1 < steps) read_b(bf[(j & 1) ^ 1], j + 1);
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][mi], bf[j & 1][ni], acc[mi][ni], 0, 0, 0);
                // (its next use: NS steps on, or the next chunk's step of the same set)
                const uint32_t src = j + NS < steps ? w_cur + (j + NS) * kStep : w_nxt + set * kStep;
                wf[set][0] = w_load(src, 0);
                wf[set][1] = w_load(src, 1);
                __builtin_amdgcn_sched_barrier(0);
            }, std::make_integer_sequence<int, steps>{});
            if (more) stage_write(smem + ((c + 1) & 1) * Sh::BUF);
            w_cur = w_nxt;
            __syncthreads();
        }
    }
    if (mt >= p.nmt || t0 >= p.Tout) return;
    float *tp = reinterpret_cast<float *>(smem) + wave * 16 * Sh::TN;
    epi.template store_private_tile<false, true>(acc, tp, lane, b, t0, mt * kTileM);
}

// Adds the nsplit parts of 16 rows x 32 steps in order and finishes them: a wavefront of its own for each of the
// kWaves x nt such pieces of a tile (with whole 16-row quarters, a quarter of the wavefronts: 11 us instead of 4 for
// 768 channels x 600 steps in four parts, too few loads in flight).
__global__ __launch_bounds__(64) void split_reduce_kernel(const ConvGemmParams p, int nt)
{
    __shared__ __align__(16) float tp[16 * 32];
    split_reduce_piece(p, nt, (int)blockIdx.x, (int)threadIdx.x, tp);
}

// ---- K = 1 (pointwise convolution: a plain GEMM  out[b] = W' . in[b]) ----------------------------
// With one tap an activation element is used for one output row tile only, so the private staging
// of conv_gemm_kernel (each wavefront its own chunk) is staging-bound and reads the activations
// once per 64 output channels.  Here the four wavefronts of a workgroup take four 64-channel row
// tiles of the same 160 time steps and share the staged activations: a workgroup tile is
// 256 channels x 160 steps, the reduction runs in stages of 128 channels ([time][channel] in LDS,
// 272-byte rows, written cooperatively by all 256 lanes with the same transposing scheme), one
// workgroup barrier per stage.  Stages form one stream across the tiles of a workgroup: stage n is
// requested during stage n-2 (two register sets), written to LDS buffer n&1 during stage n-1, and
// each wavefront reloads a weight fragment right after its use with the next stage's.  Every
// wavefront finishes its own rows (no exchange); the LDS tile of that epilogue lies in the buffer
// the tile's last stage has just used.  Packed weights: the layout of prepack_kernel (Kp = 2, tap 0).
// (The figures above are those of the shape (2, 5, 128); PwShape lists the shapes.)
// The shape of a workgroup tile: every wavefront owns MI row blocks (32 channels each) x NT time blocks and the
// reduction runs in stages of SC channels.  (2, 5, 128): 256 channels x 160 steps, 512 LDS bytes read per MFMA;
// (4, 4, 64): 512 channels x 128 steps, all 256 accumulation registers in use, 256 LDS bytes read and half the
// staging work per MFMA -- the faster one wherever its tiles fit the tensor.
template <int MI, int NT, int SC>
struct PwShape {
    static_assert(MI % 2 == 0 && SC % kChunk == 0, "whole 64-row tiles, whole chunks");
    static constexpr int kRowTiles = MI / 2;                 // 64-row tiles of the packed weights per wavefront
    static constexpr int kChunks = SC / kChunk;              // chunks of 32 channels per stage
    static constexpr int kRowBytes = SC * 2 + 16;            // 272 / 144: any 16 consecutive rows cover all banks with 16-byte reads
    static constexpr int kRows = NT * 32;                    // time steps per tile
    static constexpr int kBufBytes = kRows * kRowBytes;
    static constexpr int kPairBlocks = SC / 32;              // blocks of 16 channel pairs
    static constexpr int kItems = NT * kPairBlocks / kWaves; // staging items per lane and stage (blocks of 16 pairs x 4 time groups)
    static_assert(kItems * kWaves == NT * kPairBlocks && kItems <= 2 * kChunks, "one staging item per k-step");
    static constexpr int kEpiBytes = kWaves * 16 * kRows * (int)sizeof(float);  // the four epilogue tiles
    static constexpr bool kEpiInBuf = kEpiBytes <= kBufBytes;  // they fit the buffer the tile's last stage has used
    static constexpr size_t kLds = 2 * (size_t)kBufBytes + (kEpiInBuf ? 0 : kEpiBytes);
};

// LEN: the launch carries input lengths (a staged group may straddle the valid length of its item) or has output
// rows of any length.
template <bool LEN, int MI, int NT, int SC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void pointwise_gemm_kernel(const ConvGemmParams p)
{
    using Sh = PwShape<MI, NT, SC>;
    constexpr int TN = NT * 32, RT = Sh::kRowTiles;
    constexpr int kPwStageCh = SC, kPwChunks = Sh::kChunks, kPwRowBytes = Sh::kRowBytes, kPwBufBytes = Sh::kBufBytes;
    constexpr int kPwItems = Sh::kItems, kPB = Sh::kPairBlocks;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int T = p.Tin;                                   // row_pitch(p.Tout)
    const int nmt4 = (p.nmt + kWaves * RT - 1) / (kWaves * RT);  // workgroup row tiles
    const int nst = (p.R + kPwStageCh - 1) / kPwStageCh;   // stages per tile
    const int ncols = p.ntt * p.B;                         // time tiles of all batch items
    const int ntiles = nmt4 * ncols;
    const int G = (int)gridDim.x;
    // Which tiles a workgroup takes.  Grouped (G a multiple of 8*nmt4): the nmt4 workgroups that need
    // the same activations run on the same XCD at the same time (XCD = blockIdx % 8), so those are
    // fetched into that L2 once: workgroup x = 8*j + c takes row tile j % nmt4 of time tile
    // it*(G/nmt4) + 8*(j/nmt4) + c in its it-th turn.  Otherwise tile x + it*G, row tile fastest.
    const bool grouped = G % (8 * nmt4) == 0;
    const int per_turn = grouped ? G / nmt4 : 0;
    const int col0 = grouped ? 8 * (((int)blockIdx.x >> 3) / nmt4) + ((int)blockIdx.x & 7) : 0;
    const int my_tiles = grouped ? (col0 < ncols ? (ncols - col0 + per_turn - 1) / per_turn : 0)
                                 : ((int)blockIdx.x < ntiles ? (ntiles - (int)blockIdx.x + G - 1) / G : 0);
    const int total = my_tiles * nst;                      // stages in this workgroup's stream
    if (total == 0) return;

    const __amdgpu_buffer_rsrc_t rs_in =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)((size_t)p.B * p.R * T * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (int)p.wp_bytes, 0x00020000);
    Epilogue<NT> epi;
    epi.init(p.out, p.res, p.scale, p.shift, p.B, p.M, p.Tout, p.relu, p.len_out, p.len_out_div);

    // position in the stream: tile coordinates and stage; advanced without divisions except at a tile change
    struct Pos {
        bool valid;
        int tile, mt4, b, t0, s;  // tile: which turn of this workgroup
        int tlen;                 // valid input length of batch item b (T without lengths)
    };
    auto decode = [&](Pos &q) {  // (mt4, b, t0) of turn q.tile; wave-uniform, pinned to scalar registers
        int ntile, mt4;
        if (grouped) {
            ntile = q.tile * per_turn + col0;
            mt4 = ((int)blockIdx.x >> 3) % nmt4;
            q.valid = ntile < ncols;
        } else {
            const int tile = (int)blockIdx.x + q.tile * G;
            q.valid = tile < ntiles;
            ntile = tile / nmt4;
            mt4 = tile - ntile * nmt4;
        }
        ntile = q.valid ? ntile : 0;
        const int b = ntile / p.ntt;
        q.mt4 = __builtin_amdgcn_readfirstlane(mt4);
        q.b = __builtin_amdgcn_readfirstlane(b);
        q.t0 = __builtin_amdgcn_readfirstlane((ntile - b * p.ntt) * TN);
        q.tlen = __builtin_amdgcn_readfirstlane(clipped_len(p.len_in, b, T));
    };
    auto advance = [&](Pos &q) {
        if (++q.s == nst) {
            q.s = 0;
            q.tile += 1;
            decode(q);
        }
    };
    // ---- activations: the stage is SC/2 channel pairs x 4*NT time groups (8 steps each), cut into blocks
    // of 16 pairs x 4 groups; block kItems*wave + it is item `it` of this wavefront: lane = (group, pair), so
    // a load instruction reads 16 rows x 64 contiguous bytes and a write instruction 16 consecutive
    // dwords in each of 4 rows
    u32x4 xa0[kPwItems], xb0[kPwItems], xa1[kPwItems], xb1[kPwItems];
    auto x_load_item = [&](const Pos &q, int it, u32x4 &xa, u32x4 &xb) {
        const uint32_t soff = (uint32_t)(q.b * p.R + q.s * kPwStageCh) * (uint32_t)(T * 2);  // < 2^30: checked by the host
        const int rem = p.R - q.s * kPwStageCh;  // channels left from this stage on
        const int blk = wave * kPwItems + it;
        const int pair = (blk % kPB) * 16 + (lane & 15), tg = (blk / kPB) * 4 + (lane >> 4);
        const int t = q.t0 + 8 * tg;
        const bool ok = q.valid && t < q.tlen;  // groups that start inside the valid length (T % 8 == 0: they end inside the row)
        const uint32_t off = (uint32_t)(((2 * pair) * T + t) * 2);
        xa = __builtin_amdgcn_raw_buffer_load_b128(rs_in, (ok && 2 * pair < rem) ? off : kOutOfRange, soff, 0);
        xb = __builtin_amdgcn_raw_buffer_load_b128(rs_in, (ok && 2 * pair + 1 < rem) ? off + (uint32_t)(T * 2) : kOutOfRange, soff, 0);
    };
    auto x_load = [&](const Pos &q, u32x4(&xa)[kPwItems], u32x4(&xb)[kPwItems]) {
#pragma unroll
        for (int it = 0; it < kPwItems; ++it) x_load_item(q, it, xa[it], xb[it]);
    };
    // (time steps at or beyond the valid length of the stage's batch item are written as zeros)
    auto x_write_item = [&](unsigned char *buf, const Pos &q, int it, const u32x4 &xa, const u32x4 &xb) {
        const int blk = wave * kPwItems + it;
        const int pair = (blk % kPB) * 16 + (lane & 15), tg = (blk / kPB) * 4 + (lane >> 4);
        uint32_t *dst = reinterpret_cast<uint32_t *>(buf + (8 * tg) * kPwRowBytes + pair * 4);
        const int nvalid = q.tlen - (q.t0 + 8 * tg);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (LEN) {
                dst[(2 * j) * (kPwRowBytes / 4)] = nvalid > 2 * j ? zip_lo16(xa[j], xb[j]) : 0u;
                dst[(2 * j + 1) * (kPwRowBytes / 4)] = nvalid > 2 * j + 1 ? zip_hi16(xa[j], xb[j]) : 0u;
            } else {  // T % 8 == 0: a group lies wholly inside the row or was loaded as zeros
                dst[(2 * j) * (kPwRowBytes / 4)] = zip_lo16(xa[j], xb[j]);
                dst[(2 * j + 1) * (kPwRowBytes / 4)] = zip_hi16(xa[j], xb[j]);
            }
        }
    };
    // ---- weights of this wavefront's 32*MI rows: [chunk of the stage][ks][mi], reloaded in place
    bf16x8 wf[kPwChunks][2][MI];
    const uint32_t w_lane = (uint32_t)lane * 16;
    const uint32_t chunk_bytes = (uint32_t)p.Kp * 4 * 64 * 16;
    auto w_off = [&](const Pos &q, int j, int rt) {  // byte offset of chunk j of the stage for row tile rt of this wavefront, or out of range
        const int mt = (q.mt4 * kWaves + wave) * RT + rt, c = q.s * kPwChunks + j;
        return (q.valid && mt < p.nmt && c < p.nch) ? (uint32_t)(mt * p.nch + c) * chunk_bytes : kOutOfRange;
    };
    auto w_load = [&](uint32_t off, int f) {
        // an absent chunk: offset beyond the packed tensor (the hardware returns zeros)
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_lane + (uint32_t)f * 1024u + (off == kOutOfRange ? kOutOfRange : 0u),
                                                                                off == kOutOfRange ? 0u : off, 0));
    };

    f32x16 acc[RT][2][NT];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi >> 1][mi & 1][ni][r] = 0.f;

    // The accumulators stay in accumulation registers across stages: without these empty statements at
    // every place where the loop-carried value is defined, the allocator moves all of them to vector
    // registers and back at every loop header.
    auto pin_acc = [&]() {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) asm volatile("" : "+a"(acc[mi >> 1][mi & 1][ni]));
    };
    pin_acc();
    // ---- prologue: stage 0 into buffer 0, stage 1 into the second register set, weights of stage 0
    Pos q0, q1, q2;  // this stage, the next, the one after
    q0.tile = 0;  // turn number
    q0.s = 0;
    decode(q0);
    q1 = q0;
    advance(q1);
    q2 = q1;
    advance(q2);
    {
#pragma unroll
        for (int j = 0; j < kPwChunks; ++j)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const uint32_t o = w_off(q0, j, rt);
#pragma unroll
                for (int f = 0; f < 4; ++f) wf[j][f >> 1][2 * rt + (f & 1)] = w_load(o, f);
            }
        x_load(q0, xa0, xb0);
        x_load(q1, xa1, xb1);
#pragma unroll
        for (int it = 0; it < kPwItems; ++it) x_write_item(smem, q0, it, xa0[it], xb0[it]);
        __syncthreads();
    }
    const int lane_off = (lane & 31) * kPwRowBytes + (lane >> 5) * 16;
    // one stage: k even uses buffer 0 / requests into set 0 (whose data, stage k, is in LDS already) and
    // writes set 1 (stage k+1) into buffer 1; k odd the other way round.  (Always inlined: as a call it would have all of the
    // accumulators in scratch memory, 22 x 1024 -> 768 channels, T=490: 2163 us instead of 66.)
    auto stage = [&](unsigned char *cur, unsigned char *nxt, u32x4(&xa)[kPwItems], u32x4(&xb)[kPwItems],
                     const u32x4(&xo_a)[kPwItems], const u32x4(&xo_b)[kPwItems]) __attribute__((always_inline)) {
        const Pos q = q0;
        const unsigned char *bbase = cur + lane_off;
        bf16x8 b0[NT], b1[NT];
        pin_acc();
        auto read_b = [&](bf16x8(&dst)[NT], int j, int ks) {
#pragma unroll
            for (int ni = 0; ni < NT; ++ni)
                dst[ni] = *reinterpret_cast<const bf16x8 *>(bbase + ni * 32 * kPwRowBytes + j * 64 + ks * 32);
        };
        read_b(b0, 0, 0);
        // one k-step: MI*NT MFMAs from fragments (j, ks), which are then reloaded with the next stage's
        auto kstep = [&](int j, int ks, const bf16x8(&bc)[NT], const uint32_t(&o)[RT]) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
                    acc[mi >> 1][mi & 1][ni] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j][ks][mi], bc[ni], acc[mi >> 1][mi & 1][ni], 0, 0, 0);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) wf[j][ks][mi] = w_load(o[mi >> 1], ks * 2 + (mi & 1));
            // the writes of the next stage ride on the last k-steps (its loads are two stages old)
            constexpr int first = 2 * kPwChunks - kPwItems;
            const int step = 2 * j + ks;
            if (step < kPwItems) x_load_item(q2, step, xa[step], xb[step]);  // the stage after the next, one item per k-step
            if (step >= first) x_write_item(nxt, q1, step - first, xo_a[step - first], xo_b[step - first]);
            __builtin_amdgcn_sched_barrier(0);  // keeps every load where it is written
        };
#pragma unroll
        for (int j = 0; j < kPwChunks; ++j) {
            uint32_t o[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) o[rt] = w_off(q1, j, rt);
            read_b(b1, j, 1);
            kstep(j, 0, b0, o);
            if (j + 1 < kPwChunks) read_b(b0, j + 1, 0);
            kstep(j, 1, b1, o);
        }
        __syncthreads();  // stage k+1 is complete in LDS; buffer `cur` may be overwritten
        if (q.valid && q.s == nst - 1) {
            // the tile is finished: this wavefront's rows leave through its slice of `cur` (or of the
            // region behind the two buffers where the four slices do not fit one buffer)
            const int el = fresh_lane();
            unsigned char *ebase = Sh::kEpiInBuf ? cur : smem + 2 * kPwBufBytes;
            float *tp = reinterpret_cast<float *>(ebase + (size_t)wave * 16 * TN * sizeof(float));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                epi.template store_private_tile<false, LEN>(acc[rt], tp, el, q.b, q.t0, ((q.mt4 * kWaves + wave) * RT + rt) * kTileM);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[mi >> 1][mi & 1][ni][r] = 0.f;
            if (Sh::kEpiInBuf) __syncthreads();  // before the next stage writes into `cur`
        }
        pin_acc();
        q0 = q1;
        q1 = q2;
        advance(q2);
    };
    for (int k = 0; k < total; k += 2) {
        stage(smem, smem + kPwBufBytes, xa0, xb0, xa1, xb1);
        stage(smem + kPwBufBytes, smem, xa1, xb1, xa0, xb0);
    }
}

// ---- K = 1 with at most 32 reduction channels and no epilogue (the input gradient of a projection onto a few
// channels, 1024 -> 29 in front of the decoder): out[b][m][t] = sum_{r < R} W'[m][r] * in[b][r][t] ------------
// The arithmetic is nothing; the pass is bound by writing `out` once.  A workgroup owns 64 time steps of one
// batch item: the R x 64 strip of `in` is copied to LDS as it lies in memory (one 16-byte load per lane) and
// comes back through the transposing LDS read as the A operand (row = time step, k = reduction channel), the
// packed weights are the B operand straight from L2 (column = output channel), so an accumulator register
// holds four consecutive time steps of one output channel and a block is transposed for the stores with 8-byte
// LDS writes.  The wavefronts of the workgroups of a grid column share out the output channels in blocks of 32.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
constexpr int kFewStrip = 64;  // time steps per workgroup
constexpr int kFewRowBytes = kFewStrip * 2 + 16;  // 144: 16-byte aligned rows; 16 consecutive lanes write 16 different bank pairs
constexpr int kFewTileBytes = 32 * kFewRowBytes;  // 32 channel rows

__global__ __launch_bounds__(kThreads) void few_channels_gemm_kernel(const ConvGemmParams p)
{
    __shared__ __align__(16) unsigned char strip[4 * 1024];  // block (step s of 16 channels, 32-step half mb): 16 rows x 64 bytes
    __shared__ __align__(16) unsigned char otile[kWaves * 2 * kFewTileBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int T = p.Tout;  // == p.Tin
    const int nstrips = (T + kFewStrip - 1) / kFewStrip;
    const int b = (int)blockIdx.x / nstrips, t0 = ((int)blockIdx.x - b * nstrips) * kFewStrip;
    const __amdgpu_buffer_rsrc_t rs_in =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)((size_t)p.B * p.R * T * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (int)p.wp_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_out =
        __builtin_amdgcn_make_buffer_rsrc((void *)p.out, 0, (int)((size_t)p.B * p.M * T * 2), 0x00020000);
    {   // wavefront w copies block w: lane = (channel row lane/4, time steps 8*(lane%4) .. +7)
        const int s = wave >> 1, mb = wave & 1;
        const int r = s * 16 + (lane >> 2), t = t0 + mb * 32 + 8 * (lane & 3);
        const bool ok = r < p.R && t < T;  // T % 8 == 0: a group lies inside the row or outside
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs_in, ok ? (uint32_t)(((b * p.R + r) * T + t) * 2) : kOutOfRange, 0, 0);
        *reinterpret_cast<u32x4 *>(strip + wave * 1024 + lane * 16) = v;
    }
    __syncthreads();
    // transposing read of a block: the lane receives time step lane%32, channels 8*(lane/32) .. +7 of the step
    const int g4 = lane >> 4, i16 = lane & 15;
    const uint32_t tr_off = (uint32_t)((8 * (g4 >> 1) + (i16 >> 2)) * 64 + (16 * (g4 & 1) + 4 * (i16 & 3)) * 2);
    bf16x8 a[2][2];  // [mb][ks]
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            union {
                s16x4 h[2];
                bf16x8 v;
            } cvt;
            const unsigned char *q = strip + (ks * 2 + mb) * 1024 + tr_off;
            cvt.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(q));
            cvt.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(q + 4 * 64));
            a[mb][ks] = cvt.v;
        }
    // blocks of 32 output channels of this wavefront
    const int nblocks = (p.M + 31) >> 5, nshare = kWaves * (int)gridDim.y, per = (nblocks + nshare - 1) / nshare;
    const int nb0 = ((int)blockIdx.y * kWaves + wave) * per, nb1 = min(nblocks, nb0 + per);
    const uint32_t chunk_bytes = (uint32_t)p.Kp * 4 * 64 * 16;  // one 64-row tile of the packed weights (R <= 32: one chunk)
    auto load_w = [&](int nb, int ks) {  // fragment (ks, mi = nb % 2) of tap 0 of row tile nb / 2; beyond the range: zeros
        const uint32_t off = (uint32_t)(nb >> 1) * chunk_bytes + (uint32_t)(ks * 2 + (nb & 1)) * 1024u;
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_w, nb < nb1 ? (uint32_t)lane * 16 : kOutOfRange,
                                                                                nb < nb1 ? off : 0u, 0));
    };
    // The result block (32 output channels x 64 time steps) goes through a wave-private LDS tile, [channel][time]
    // in bf16 with rows of 144 bytes, so that it leaves in 16-byte stores whose lanes run along the row: a request to L2 per 64 bytes instead of one per
    // 8 (at one request per lane the pass was bound by the request rate, not by the bytes).  Two tiles in turn.
    unsigned char *tiles = otile + wave * 2 * kFewTileBytes;
    const int h = lane >> 5;
    auto block = [&](int nb, const bf16x8(&w)[2], int par) {
        if (nb >= nb1) return;
        unsigned char *tile = tiles + par * kFewTileBytes;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mb][0], w[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mb][1], w[1], acc, 0, 0, 0);
            // registers 4j .. 4j+3: time steps 32*mb + 8*j + 4*h .. +3 of output channel lane % 32
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u32x2 o = {pack_bf16x2(acc[4 * j], acc[4 * j + 1]), pack_bf16x2(acc[4 * j + 2], acc[4 * j + 3])};
                *reinterpret_cast<u32x2 *>(tile + (lane & 31) * kFewRowBytes + (32 * mb + 8 * j + 4 * h) * 2) = o;
            }
        }
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // item: (channel row, 8 time steps)
            const int idx = lane + 64 * i, row = idx >> 3, piece = idx & 7;
            const int m = nb * 32 + row, t = t0 + 8 * piece;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(tile + row * kFewRowBytes + piece * 16);
            const bool ok = m < p.M && t < T;  // T % 8 == 0
            __builtin_amdgcn_raw_buffer_store_b128(v, rs_out, ok ? (uint32_t)(((b * p.M + m) * T + t) * 2) : kOutOfRange, 0, 0);
        }
    };
    bf16x8 w0[2] = {load_w(nb0, 0), load_w(nb0, 1)}, w1[2] = {load_w(nb0 + 1, 0), load_w(nb0 + 1, 1)};
    for (int nb = nb0; nb < nb1; nb += 2) {
        block(nb, w0, 0);
        w0[0] = load_w(nb + 2, 0);
        w0[1] = load_w(nb + 2, 1);
        block(nb + 1, w1, 1);
        w1[0] = load_w(nb + 3, 0);
        w1[1] = load_w(nb + 3, 1);
        wave_lds_fence();  // the reads of both tiles are done before the next pair of blocks writes them
    }
}

// Packed weights: [mt][chunk][tap < Kp][ks][mi][lane][8] (Kp = K rounded up to even, the extra
// tap is zero); element (lane, j) of fragment (ks, mi) is
// W'[m = mt*64 + mi*32 + lane%32][r = chunk*32 + ks*16 + 8*(lane/32) + j][tap], zero outside,
// with W'[m][r][k] = w[m][r][k] (forward) or w[r][m][K-1-k] * rscale[r] (input gradient: FLIP; r is the
// block's output channel co, rscale its folded-BatchNorm factor or NULL for 1; the product is rounded to
// bf16, so the input gradient contracts the exact dy*[y>0] with bf16(w*scale)).
// One block packs 16 of the 64 channels of one (mt, chunk): it copies that 16x32xK block of w
// into LDS with coalesced reads (runs of 32*K, resp. 16*K, contiguous elements) and gathers the
// fragments from there.
constexpr int kPackRows = 16;
// elements between consecutive channels m of the LDS tile: 32*K plus one dword of padding, which
// makes the stride an odd number of dwords so that lanes with different m hit different banks
__host__ __device__ constexpr int pack_m_stride(int K) { return kChunk * K + 2; }
// The two parities' filters of a stride-2 input gradient, as one filter with twice the output rows (see there).
struct Phases {
    int K, padL;            // taps and left padding of the joint contraction
    int kp[2], Kr[2], off[2];  // parity r: taps kp, kp+2, ... (Kr of them) lie at off .. of its filter
    int U, Up;              // outputs per parity, row pitch
    bool ok;
};
// PHASES: M = 2*Cin rows (parity, ci) of taps cut out of w, which is [R][Cin][ld] here (FLIP).
template <bool FLIP, bool PHASES = false>
__device__ __forceinline__ void prepack_block(unsigned blk, unsigned char *smem, const bf16_t *__restrict__ w,
                                              u32x4 *__restrict__ wp, int M, int R, int K, int nch,
                                              int ld /* row length of w */, size_t zero_off, int vec /* 16-byte aligned runs */,
                                              const float *__restrict__ rscale = nullptr, const Phases &ph = Phases{})
{
    bf16_t *tile = reinterpret_cast<bf16_t *>(smem);  // [16 m][32 r][K] as m*ms + r*K + k
    const int ms = pack_m_stride(K);
    if (blk == 0)  // one tap pair of zero weights after the packed tensor
        for (int i = threadIdx.x; i < 512; i += 256) wp[zero_off + i] = u32x4{0u, 0u, 0u, 0u};
    const int q = blk & 3;                      // which 16 channels of the 64
    const int c = (blk >> 2) % nch, mt = (blk >> 2) / nch;
    const int m0 = mt * kTileM + q * kPackRows, r0 = c * kChunk;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // Copy the block of w into LDS.  Rows of w that start on a 16-byte boundary (vec != 0) are read
    // with 16-byte buffer loads, four per thread in flight (the copy is latency bound otherwise);
    // elements beyond the tensor read zeros, elements of a neighbouring block are masked.
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)w, 0, (int)((size_t)M * R * K * 2), 0x00020000);
    const int nrows = FLIP ? kChunk : kPackRows;            // runs of contiguous elements: one per r, resp. per m
    const int run = (FLIP ? kPackRows : kChunk) * K;        // elements per run (a multiple of 8)
    const int valid = FLIP ? max(0, min(kPackRows, M - m0)) * K : max(0, min(kChunk, R - r0)) * K;
    auto row_ok = [&](int row) { return FLIP ? r0 + row < R : m0 + row < M; };
    auto row_off = [&](int row) {  // element offset of the run in w
        return FLIP ? (size_t)(r0 + row) * ld + (size_t)m0 * K : (size_t)(m0 + row) * ld + (size_t)r0 * K;
    };
    auto row_factor = [&](int row) {  // FLIP only: a run belongs to one reduction channel
        return (FLIP && rscale && r0 + row < R) ? rscale[r0 + row] : 1.f;
    };
    const bool scaled = FLIP && rscale != nullptr;
    auto put = [&](int row, int o, bf16_t v, float f) {  // element o of run `row`
        if (FLIP) {
            const int m = o / K, k = o - m * K;
            tile[m * ms + row * K + (K - 1 - k)] = scaled ? f32_to_bf16(bf16_to_f32(v) * f) : v;
        } else {
            tile[row * ms + o] = v;
        }
    };
    if constexpr (PHASES) {
        const int Cin = M / 2;
        for (int o0 = threadIdx.x; o0 < nrows * run; o0 += 256 * 4) {
            bf16_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int o = o0 + u * 256, row = o / run, m = m0 + (o - row * run) / K, k = (o - row * run) % K;
                const int r = m >= Cin ? 1 : 0, tap = k - ph.off[r];
                const bool ok = o < nrows * run && row_ok(row) && m < M && tap >= 0 && tap < ph.Kr[r];
                v[u] = ok ? w[((size_t)(r0 + row) * Cin + m - r * Cin) * ld + ph.kp[r] + 2 * tap] : (bf16_t)0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int o = o0 + u * 256, row = o / run;
                if (o < nrows * run) put(row, o - row * run, v[u], row_factor(row));
            }
        }
    } else if (vec) {
        const int vpr = run / 8, nvec = nrows * vpr;
        for (int v0 = threadIdx.x; v0 < nvec; v0 += 256 * 4) {
            u32x4 d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int v = v0 + u * 256;
                const int row = v / vpr, o = (v - row * vpr) * 8;
                const bool ok = v < nvec && row_ok(row) && o < valid;
                d[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? (uint32_t)((row_off(row) + o) * 2) : 0x80000000u, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int v = v0 + u * 256;
                if (v < nvec) {
                    const int row = v / vpr, o = (v - row * vpr) * 8;
                    const float f = row_factor(row);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint32_t word = d[u][e >> 1];
                        const bf16_t val = (bf16_t)((e & 1) ? word >> 16 : word & 0xffffu);
                        put(row, o + e, (o + e < valid) ? val : (bf16_t)0, f);
                    }
                }
            }
        }
    } else {
        for (int row = wv; row < nrows; row += 4) {
            const bool ok = row_ok(row);
            const bf16_t *src = w + (ok ? row_off(row) : (size_t)0);
            const float f = row_factor(row);
            for (int o = lane; o < run; o += 64) put(row, o, (ok && o < valid) ? src[o] : (bf16_t)0, f);
        }
    }
    __syncthreads();
    const int Kp = (K + 1) & ~1;  // an odd K gets one zero tap
    u32x4 *dst = wp + (size_t)(blk >> 2) * Kp * 256;
    const int mi = q >> 1, lane_lo = (q & 1) * 16;
    for (int idx = threadIdx.x; idx < Kp * 64; idx += 256) {
        const int m16 = idx & 15, half = (idx >> 4) & 1, ks = (idx >> 5) & 1, k = idx >> 6;
        u32x4 out = {0u, 0u, 0u, 0u};
        if (k < K) {
            const bf16_t *src = tile + m16 * ms + (ks * 16 + 8 * half) * K + k;
#pragma unroll
            for (int j = 0; j < 4; ++j) out[j] = (uint32_t)src[(2 * j) * K] | ((uint32_t)src[(2 * j + 1) * K] << 16);
        }
        dst[(k * 4 + ks * 2 + mi) * 64 + half * 32 + lane_lo + m16] = out;
    }
}

template <bool FLIP>
__global__ __launch_bounds__(256) void prepack_kernel(const bf16_t *__restrict__ w, u32x4 *__restrict__ wp, int M,
                                                      int R, int K, int nch, int ld, size_t zero_off, int vec,
                                                      const float *__restrict__ rscale)
{
    extern __shared__ __align__(16) unsigned char smem[];
    prepack_block<FLIP>(blockIdx.x, smem, w, wp, M, R, K, nch, ld, zero_off, vec, rscale);
}

// Everything the input-gradient engine needs, in one launch: the first npack blocks pack the
// flipped weights times the affine factor of their output channel (a latency-bound job), the others
// run the elementwise mask pass g = dy*[y>0] (bandwidth bound), so the two overlap instead of
// following each other.  g is what the engine contracts; it is also the residual gradient, so it
// is written straight into dres when the caller asked for that, into the workspace otherwise.
__global__ __launch_bounds__(256) void dgrad_prepare_kernel(unsigned npack, const bf16_t *__restrict__ w,
                                                            u32x4 *__restrict__ wp, int M, int R, int K, int nch,
                                                            int ld, size_t zero_off, int vec,
                                                            const float *__restrict__ rscale, size_t n8,
                                                            const u32x4 *__restrict__ dy, const u32x4 *__restrict__ y,
                                                            int relu, u32x4 *__restrict__ gout)
{
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x < npack) {
        prepack_block<true>(blockIdx.x, smem, w, wp, M, R, K, nch, ld, zero_off, vec, rscale);
    } else {
        const size_t i = (size_t)(blockIdx.x - npack) * 256 + threadIdx.x;
        if (i < n8) gout[i] = relu ? masked_grad8(dy[i], y[i]) : dy[i];
    }
}

// The same for a fused backward call: the elementwise part also writes g in the fragment order
// of the stride-1 weight-gradient kernels (mask_pack_wave), so dy and y are read once for both gradients.
// gplain may be NULL (no ReLU and no residual gradient wanted: the engine then reads dy itself).
__global__ __launch_bounds__(256) void bwd_prepare_kernel(unsigned npack, const bf16_t *__restrict__ w,
                                                          u32x4 *__restrict__ wp, int M, int R, int K, int nch, int ld,
                                                          size_t zero_off, int vec, const float *__restrict__ rscale,
                                                          int B, int Cout, int To, int ncm, int nst,
                                                          const bf16_t *__restrict__ dy, const bf16_t *__restrict__ y,
                                                          int relu, u32x4 *__restrict__ gplain, u32x4 *__restrict__ gf)
{
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x < npack) {
        prepack_block<true>(blockIdx.x, smem, w, wp, M, R, K, nch, ld, zero_off, vec, rscale);
        return;
    }
    const unsigned nst4 = (unsigned)(nst + 3) / 4;
    const unsigned item = (blockIdx.x - npack) * 4 + (threadIdx.x >> 6);  // (b, cm, st4), st4 fastest
    if (item >= (unsigned)B * ncm * nst4) return;
    const int st4 = item % nst4, cm = (item / nst4) % ncm, b = item / (nst4 * ncm);
    mask_pack_wave(threadIdx.x & 63, b, cm, st4, Cout, To, ncm, nst, dy, y, relu, gplain, gf);
}

// ---- stride-2 input gradient --------------------------------------------------------------------
// dx[ci][2u + r] only receives the taps k with 2u + r + pad - k even, so each parity r of the sample is a stride-1
// correlation of g with every second tap.  The two are one contraction with 2*Cin output rows (parity, ci): their
// filters are cut out of w while they are packed (prepack_block), side by side and aligned to the same window with zero taps
// where they differ, and interleave_phases_kernel merges the rows.  64 <- 256 channels, K=11, B=32, T=1600: one contraction over shared windows
// in place of one per parity.
// dx[b][ci][2u + r] = a[b][r][ci][u], zero from a sample's length on; eight samples per thread, rows of any length.
// A NaN may come from a zero tap times an infinite gradient: it is made again from the products the definition has (an
// infinite gradient would else leave NaNs in samples that no tap connects to it).
struct PhaseSums {
    int Cout, To, K, pad, pitch;  // pitch of g
    const bf16_t *g, *w;
    const float *scale;
};
__device__ __forceinline__ bf16_t defined_dx(const PhaseSums &q, int Cin, unsigned b, unsigned ci, int tau)
{
    float z = 0.f;
#pragma clang loop unroll(disable)
    for (int co = 0; co < q.Cout && z == z; ++co) {
        const bf16_t *g = q.g + ((size_t)b * q.Cout + co) * q.pitch, *w = q.w + ((size_t)co * Cin + ci) * q.K;
#pragma clang loop unroll(disable)
        for (int k = (tau + q.pad) & 1; k < q.K; k += 2) {
            const int t = (tau + q.pad - k) >> 1;
            if (t < 0 || t >= q.To) continue;
            z = fmaf(q.scale ? bf16_to_f32(f32_to_bf16(bf16_to_f32(w[k]) * q.scale[co])) : bf16_to_f32(w[k]), bf16_to_f32(g[t]), z);
        }
    }
    return f32_to_bf16(z);
}
__global__ __launch_bounds__(256) void interleave_phases_kernel(const bf16_t *__restrict__ a, bf16_t *__restrict__ dx, int Cin, int T,
                                                                int Up, unsigned n, const int *__restrict__ len, const PhaseSums q)
{
    const unsigned i = blockIdx.x * 256 + threadIdx.x;
    const unsigned T8 = (unsigned)(T + 7) / 8;
    if (i >= n) return;
    const unsigned row = i / T8, grp = i - row * T8, b = row / (unsigned)Cin, ci = row - b * (unsigned)Cin;
    const bf16_t *e = a + ((size_t)(2 * b) * Cin + ci) * Up + 4 * grp;
    uint32_t ev[2], ov[2];
    __builtin_memcpy(ev, e, 8);
    __builtin_memcpy(ov, e + (size_t)Cin * Up, 8);
    u32x4 v = {zip_lo16(ev[0], ov[0]), zip_hi16(ev[0], ov[0]), zip_lo16(ev[1], ov[1]), zip_hi16(ev[1], ov[1])};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int tau = 8 * (int)grp + 2 * j;
        if ((v[j] & 0x7fffu) > 0x7f80u && tau < T) v[j] = (v[j] & 0xffff0000u) | defined_dx(q, Cin, b, ci, tau);
        if ((v[j] >> 16 & 0x7fffu) > 0x7f80u && tau + 1 < T)
            v[j] = (v[j] & 0xffffu) | (uint32_t)defined_dx(q, Cin, b, ci, tau + 1) << 16;
    }
    if (len) {
        const int nv = len[b] - 8 * (int)grp;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] &= nv >= 2 * j + 2 ? 0xffffffffu : (nv == 2 * j + 1 ? 0x0000ffffu : 0u);
    }
    store8_any(dx + (size_t)row * T + 8 * grp, v, T - 8 * (int)grp);
}

// The preparation of a call on rows that are no multiple of eight long (RowPrep): packing blocks, mask blocks (a
// wavefront per 32 channels x 64 time steps), copy blocks (a 16-byte group of the pitched copy per thread).
// Bound by memory: a 16 x 384 x 777 padded batch (K = 13, with residual) takes 201 us for the forward
// pass and both gradients, 30 900 us on the plain kernels that served such rows before.
struct PrepareRowsArgs {
    unsigned npack, nmask;
    const bf16_t *w;
    u32x4 *wp;
    int M, R, K, nch, ld, vec;
    size_t zero_off;
    const float *rscale;
    int B, Cout, To, ncm, nst, nst4, relu;
    const bf16_t *dy, *y;
    bf16_t *gplain, *dres;
    u32x4 *gf;
    int Cin, T, T8;
    size_t ngroups;
    const int *len;
    const bf16_t *x;
    u32x4 *xp;
};
template <bool FLIP>
__global__ __launch_bounds__(256) void prepare_rows_kernel(const PrepareRowsArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned blk = blockIdx.x;
    if (blk < a.npack) {
        prepack_block<FLIP>(blk, smem, a.w, a.wp, a.M, a.R, a.K, a.nch, a.ld, a.zero_off, a.vec, a.rscale);
        return;
    }
    blk -= a.npack;
    if (blk < a.nmask) {
        const unsigned item = blk * 4 + (threadIdx.x >> 6);  // (b, cm, st4), st4 fastest
        if (item >= (unsigned)(a.B * a.ncm * a.nst4)) return;
        const int st4 = item % a.nst4, cm = (item / a.nst4) % a.ncm, b = item / (a.nst4 * a.ncm);
        mask_pack_wave_any(threadIdx.x & 63, b, cm, st4, a.Cout, a.To, a.ncm, a.nst, a.dy, a.y, a.relu, a.gplain, a.dres, a.gf);
        return;
    }
    const size_t i = (size_t)(blk - a.nmask) * 256 + threadIdx.x;
    if (i >= a.ngroups) return;
    const size_t row = i / (unsigned)a.T8;
    const int t = 8 * (int)(i - row * (unsigned)a.T8);
    int n = a.T;
    if (a.len) {
        const int l = a.len[row / (unsigned)a.Cin];
        n = l < 0 ? 0 : (l < n ? l : n);
    }
    if (a.T >= 8)
        a.xp[i] = first_of8(shift8_down(load8_row(a.x + row * a.T, t, a.T), t, a.T), n - t);
    else
        a.xp[i] = load8_any(a.x + row * a.T + t, n - t);
}

// A stride-2 input gradient's: the parities' filters (M = 2*Cin rows cut out of w [R][Cin][ld]) and the pass over dy and y
// for rows of any length, side by side (one after the other they took 7.3 and 6.7 us, 64 -> 256 channels, B=32, T=1600).
__global__ __launch_bounds__(256) void prepare_phases_kernel(const PrepareRowsArgs a, const Phases ph)
{
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x < a.npack) {
        prepack_block<true, true>(blockIdx.x, smem, a.w, a.wp, a.M, a.R, ph.K, a.nch, a.ld, a.zero_off, 0, a.rscale, ph);
        return;
    }
    const unsigned item = (blockIdx.x - a.npack) * 4 + (threadIdx.x >> 6);
    if (item >= (unsigned)(a.B * a.ncm * a.nst4)) return;
    const int st4 = item % a.nst4, cm = (item / a.nst4) % a.ncm, b = item / (a.nst4 * a.ncm);
    mask_pack_wave_any(threadIdx.x & 63, b, cm, st4, a.Cout, a.To, a.ncm, a.nst, a.dy, a.y, a.relu, a.gplain, a.dres, nullptr);
}

struct Plan {
    bool ok;
    int nt;       // NT template value (5 or 2)
    int stride;   // 1 or 2
    int nitems;   // staging items per lane; a buffer holds nitems*32 + kDumpRows rows
    int buf_bytes;
    int overlap;  // cross-tile staging possible
    bool unrolled;  // the kernel instance with an unrolled chunk for this K applies
    size_t lds;
};

// Tin, Tout: lengths of the rows that are staged / written; the staged ones must be 16-byte aligned (% 8 == 0).
// R: reduction channels (cross-tile staging needs every wavefront to own the same number of chunks).
Plan make_plan(int Tin, int Tout, int R, int K, int stride, int dil)
{
    Plan pl = {};
    pl.stride = stride;
    if (stride != 1 && stride != 2) return pl;
    if (Tin % 8 != 0) return pl;
    if ((size_t)kPackRows * pack_m_stride(K) * sizeof(bf16_t) > (size_t)kMaxLds) return pl;  // weight packing tile
    const int nch = (R + kChunk - 1) / kChunk;
    // candidate 0: the kernel with an unrolled chunk (tap counts it is built for, stride 1, wide tile,
    // equal chunk counts for the four wavefronts); it skips the zero tap of an odd K, so its window
    // counts K taps.  Candidates 1, 2: the tap-pair loop with the wide, then the narrow tile.
    for (int ci = 0; ci < 3; ++ci) {
        const bool unrolled = ci == 0;
        const int nt = ci == 2 ? 2 : 5;
        if (nt == 5 && (Tout <= 64 || stride == 2)) continue;  // short sequences: the narrow tile wastes less; stride 2: its window fits no LDS
        if (unrolled && !(stride == 1 && unrolled_slots(K) > 0 && nch % kWaves == 0)) continue;
        const long taps = unrolled ? K : (K + 1) & ~1;  // the tap-pair loop also reads the zero tap of an odd K
        const long rows = (long)(nt * 32 - 1) * stride + (taps - 1) * dil + 1 + 7;
        const long nitems = ((rows + 7) / 8 * 16 + 63) / 64;
        if (unrolled && nitems > unrolled_slots(K)) continue;
        const size_t buf = (size_t)(nitems * 32 + kDumpRows) * kRowBytes;
        const size_t stage = (size_t)kWaves * 2 * buf;
        const size_t round_bytes = (size_t)kWaves * 3 * nt * 64 * sizeof(f32x4);  // one row of blocks per round
        // with cross-tile staging the scratch must fit in the buffers of one parity
        const bool overlap = (nch % kWaves == 0) && (kWaves * buf >= round_bytes);
        const size_t lds = stage > round_bytes ? stage : round_bytes;
        if (unrolled && !overlap) continue;
        if (lds <= (size_t)kMaxLds && buf >= (size_t)16 * nt * 32 * sizeof(float)) {  // buf also holds the output transpose tile
            pl.ok = true;
            pl.nt = nt;
            pl.nitems = (int)nitems;
            pl.buf_bytes = (int)buf;
            pl.overlap = overlap ? 1 : 0;
            pl.unrolled = unrolled;
            pl.lds = lds;
            return pl;
        }
    }
    return pl;
}

// ---- which calls take conv_split_kernel ---------------------------------------------------------
// Its time and the other engines' are estimated in microseconds from measured rates (256 CUs assumed: the workspace
// query has no device).  A wavefront's MFMA costs 18 ns in the unrolled engine, 20.5 ns here with two or more workgroups
// per CU; a chunk costs 0.3 us more there for staging and the barrier (27 ns and 0.8 us alone on the CU), parts
// 6 us for the second launch and 0.42 us per MB of float32 outputs and part.  Against another engine a call in parts counts
// for 15 us at least: its third launch is bound by the host below that (called from Python, 256 channels, K=11, 200 steps take
// 20.5 us in parts, 19.1 in the other engine, though the device needs 12 and 19).  Plans that tie at the floor
// are ranked by what they take on the device (fitted to 250 geometries; the launches' replays in a graph).  Device time of a
// forward call with its weight packing, the plan taken / best plan / other engine: 768 channels K=25, 600 steps, B=1
// 40 / 40 / 66 us, B=2 54 / 54 / 66, B=4 77 (the other engine) / 82 / 77; 384 channels K=13, 600 steps 17.3 / 17.3 / 27.2;
// 512 channels K=17, 400 steps, B=4 35 / 33 / 39; 768 channels K=1, 600 steps 17.9 / 17.2 / 26.2; 512 channels K=1, 400 steps,
// B=4 21 (the other engine) / 14.6 / 21; 64 -> 256 channels, stride 2, 1600 steps, B=32 28.6 / 26.9 / 43.4; 64 -> 896
// channels K=1, 1496 steps, B=23 41 (the other engine) / 54 / 41.
// nm_conv1d_block_fwd_static promises the bits of nm_conv1d_block_fwd and has a fixed array.  So the plan of a call with the
// workspace it asked for has no more parts than kSplitRounds times what that array has left behind the weights, and the
// static call makes its columns in as many rounds.  Other calls with less room take the best plan within it.
constexpr int kSplitRounds = 4;
struct SplitPlan {
    int nt, nsplit, ngroups;  // nt = 0: another engine
    double gain;              // estimated, against that
    double device;            // estimated time on the device
    size_t lds, part_bytes, col_bytes;  // parts of all columns, of one
};

// launches in which `cols` columns are made whose parts take col_bytes each, with room for `room` bytes of them
unsigned split_rounds(unsigned cols, size_t col_bytes, size_t room)
{
    const size_t fit = room / col_bytes;
    return fit == 0 ? ~0u : (unsigned)((cols + fit - 1) / fit);
}

// Padded work of a shape: MFMAs of all its tiles over the MFMAs of the contraction, times the rounds the
// workgroups need over the rounds a perfectly divisible launch would need.
template <int MI, int NT>
double pointwise_waste(const ConvGemmParams &p, int cus)
{
    const int rows = kWaves * MI * 32, cols = NT * 32;
    const long tr = (p.M + rows - 1) / rows, tc = (p.Tout + cols - 1) / cols;
    const long tiles = tr * tc * p.B;
    const double pad = (double)(tr * rows) * (double)(tc * cols) / ((double)p.M * p.Tout);
    const double rounds = (double)((tiles + cus - 1) / cus) * cus / (double)tiles;
    return pad * rounds;
}

bool pointwise_big_tile(const ConvGemmParams &p, int cus)
{
    // the 512 x 128 tile does half the LDS and staging work per MFMA and has half as many epilogue rounds per
    // output (measured 1.1 to 1.2 times faster per MFMA issued at 896 <-> 1024 channels); it is taken unless
    // its padding and last-round losses outweigh that
    return pointwise_waste<4, 4>(p, cus) <= 1.12 * pointwise_waste<2, 5>(p, cus);
}

// Pointwise layers of whole tiles and chunks have estimates of their own, fitted to all plans of 101 forward calls (256 to 1024
// channels, 56 to 13000 steps; on the device, tensors that no cache holds, weight packing left out; rms 6.5 %).  The plan
// taken is 1.9 % from the fastest on average, 7.4 % by the rates of the other calls, which hold parts too dear and the large
// kernels too cheap: 512 -> 640 channels, B=1, T=600: pointwise_gemm_kernel 22.8 us, two parts 16.5; 896 -> 1024, B=1, T=56: tap-pair
// kernel 19.9, parts 14.8.  Two workgroups share a CU from the 257th on.
bool whole_pointwise(const Plan &pl, int M, int R, int K)
{
    return K == 1 && pl.stride == 1 && M >= 256 && R >= 256 && M % kTileM == 0 && R % kChunk == 0;
}
double layer_split_cost(int nt, int ns, unsigned wgs, unsigned chunks, double mb)
{
    const unsigned last = wgs % 512, pairs = wgs / 512 + (last > 256 ? 1 : 0);
    const double one = last > 0 && last <= 256 ? (0.155 + 0.162 * nt) * chunks - 0.95 : 0.0;
    return 8.5 + one + pairs * ((0.136 + 0.141 * nt) * chunks + 0.5) + 0.46 * mb + (ns > 1 ? 1.3 + 0.5 * ns * mb : 0.0);
}
double layer_engine_cost(const Plan &pl, int B, int M, int R, int Tout)
{
    const long cus = 256;
    const int nmt = M / kTileM;
    const double base = 6.2 + 0.26 * 4e-6 * B * M * (double)Tout;
    if (pl.nt != 5) {
        const long tiles = (long)nmt * ((Tout + pl.nt * 32 - 1) / (pl.nt * 32)) * B;
        return base + (double)((tiles + cus - 1) / cus) * 1.47 * ((R + 127) / 128);
    }
    ConvGemmParams p = {};
    p.M = M; p.B = B; p.Tout = Tout;
    const bool big = pointwise_big_tile(p, cus);
    const long tiles = big ? (long)((nmt + 7) / 8) * ((Tout + 127) / 128) * B : (long)((nmt + 3) / 4) * ((Tout + 159) / 160) * B;
    const double tile = big ? 1.75 * ((R + 63) / 64) + 0.1 : 1.83 * ((R + 127) / 128) + 6.9;
    return base + (double)((tiles + cus - 1) / cus) * (tile + (Tout % 8 != 0 ? 4.7 : 0.0));  // (that instance's epilogue)
}

double engine_cost(const Plan &pl, int B, int M, int R, int Tout, int K)
{
    const long cus = 256;
    const int nmt = (M + kTileM - 1) / kTileM, nch = (R + kChunk - 1) / kChunk;
    if (K == 1 && nmt >= 2 && pl.nt == 5 && pl.stride == 1) {  // pointwise_gemm_kernel, its two tiles
        const long tiles = (long)((nmt + 3) / 4) * ((Tout + 159) / 160) * B;
        const long tiles_big = (long)((nmt + 7) / 8) * ((Tout + 127) / 128) * B;
        const double a = (double)((tiles + cus - 1) / cus) * (3.0 * ((R + 127) / 128) + 4.0);
        const double c = (double)((tiles_big + cus - 1) / cus) * (1.7 * ((R + 63) / 64) + 2.5);
        return a < c ? a : c;
    }
    const long tiles = (long)nmt * ((Tout + pl.nt * 32 - 1) / (pl.nt * 32)) * B;
    const long grid = tiles < cus ? tiles : cus;
    const double chunk = 0.018 * 4 * pl.nt * (pl.unrolled ? K : (K + 1) & ~1);
    const long full = pl.unrolled ? tiles / (kWaves * grid) + (tiles % (kWaves * grid) > 2 * grid ? 1 : 0) : 0;
    const long left = tiles - full * kWaves * grid;
    const long shared = left > 0 ? (left + grid - 1) / grid : 0;
    return full * (nch * chunk + 2.0) + shared * (((nch + kWaves - 1) / kWaves) * chunk + 4.0);
}

// part_limit: room for the parts of a round, of at most `most_rounds`
SplitPlan make_split_plan(const Plan &pl, int B, int M, int R, int Tout, int K, int dil, size_t part_limit, unsigned most_rounds)
{
    SplitPlan best = {};
    const int nmt = (M + kTileM - 1) / kTileM, nch = (R + kChunk - 1) / kChunk;
    if (!pl.ok || (K == 1 && nch == 1)) return best;
    const double mb = 4e-6 * B * M * (double)Tout;
    const bool layer = whole_pointwise(pl, M, R, K);
    // (a tie with another engine goes to that)
    double best_cost = layer ? 0.96 * layer_engine_cost(pl, B, M, R, Tout) : 0.9 * engine_cost(pl, B, M, R, Tout, K), best_on_device = 0.0;
    // (whatever the shape, the MFMAs at 256 CUs' full rate: most large calls need not be looked at any further)
    if (0.0205 / 4096 * nmt * 2 * (double)B * ((Tout + 31) / 32) * nch * 2 * K > best_cost) return best;
    for (int nt = pl.stride == 1 ? 4 : 3; nt >= 2; --nt) {
        const long rows = (long)(nt * 32 - 1) * pl.stride + (long)(K - 1) * dil + 1 + 7;
        if (rows > kSplitRows) continue;
        const long tiles_l = (long)nmt * ((Tout + nt * 32 - 1) / (nt * 32)) * B;
        if (tiles_l > (1 << 20)) continue;
        const unsigned tiles = (unsigned)tiles_l;
        for (const int ns : {1, 2, 3, 4, 6, 8, 12, 16}) {
            const unsigned wgs = tiles * ns, rounds = (wgs + 255) / 256;
            if (ns > nch || (ns > 1 && wgs > 1024)) break;
            const unsigned chunks = (unsigned)(nch + ns - 1) / (unsigned)ns;
            double cost = (double)(rounds * chunks) *
                          ((rounds > 1 ? 0.0205 : 0.027) * ((K + 1) / 2) * 2 * nt + (rounds > 1 ? 0.3 : 0.8));
            if (ns > 1) cost = std::max(cost + 6.0 + 0.42 * ns * mb, 15.0);
            if (layer) cost = layer_split_cost(nt, ns, wgs, chunks, mb);
            const double on_device = (double)(rounds * chunks) *
                                         ((rounds > 1 ? 0.026 : 0.032) * ((K + 1) / 2) * 2 * nt + (rounds > 1 ? 0.25 : 0.62)) +
                                     0.78 * rounds + 1.4 + 0.79 * ns * mb;
            if (cost > best_cost || (cost == best_cost && on_device >= best_on_device)) continue;
            const size_t col_bytes = ns > 1 ? (size_t)nmt * ns * kTileM * nt * 32 * sizeof(float) : 0;
            if (col_bytes > 0 && split_rounds(wgs / (unsigned)(nmt * ns), col_bytes, part_limit) > most_rounds) continue;
            best_cost = cost;
            best_on_device = on_device;
            best.device = on_device;
            best.gain = engine_cost(pl, B, M, R, Tout, K) - cost;
            best.nt = nt;
            best.nsplit = ns;
            best.ngroups = (int)((rows + 7) / 8);
            const size_t stage = 2 * (size_t)best.ngroups * 8 * kRowBytes;
            const size_t red = (size_t)kWaves * 3 * nt * 64 * sizeof(f32x4);
            best.lds = stage > red ? stage : red;
            best.col_bytes = col_bytes;
            best.part_bytes = align_up(wgs / (unsigned)(nmt * ns) * col_bytes, 256);
        }
    }
    return best;
}

// the same, remembered: a call asks several times (workspace query, checks, launch)
constexpr size_t kNoLimit = (size_t)1 << 38;  // (its number of 256-byte units is a key of the table below, an int)
SplitPlan split_plan(const Plan &pl, int B, int M, int R, int Tout, int K, int dil, size_t part_limit = kNoLimit, unsigned most_rounds = 1)
{
    struct Entry {
        int key[12];
        SplitPlan plan;
    };
    static thread_local Entry table[16] = {};  // (no call has B = 0)
    part_limit = std::min(part_limit, kNoLimit) >> 8 << 8;
    const int key[12] = {B, M, R, Tout, K, dil, pl.stride, pl.nt, pl.ok, pl.unrolled, (int)(part_limit >> 8), (int)most_rounds};
    unsigned h = 0;
    for (int k : key) h = h * 31u + (unsigned)k;
    Entry &t = table[(h ^ (h >> 7) ^ (h >> 15)) % 16];
    if (memcmp(t.key, key, sizeof key) != 0) {
        t.plan = make_split_plan(pl, B, M, R, Tout, K, dil, part_limit, most_rounds);
        memcpy(t.key, key, sizeof key);
    }
    return t.plan;
}

// What a call on packed weights takes on the device, packing included (fitted to the 345 geometries of unpacked_plan; rms 7 %):
// the engines' own estimates above, corrected, a launch of the packing (an input gradient's has a pass over dy in it that
// stays), its bytes and, forward, a copy of rows that are no multiple of eight long.
double packed_cost(const Plan &pl, const SplitPlan &sp, int B, int M, int R, int Tin, int Tout, int K, bool flip)
{
    const double w = 2e-6 * M * R * K;
    const double run = sp.nt ? 5.8 + 0.73 * sp.device : 3.7 + 0.99 * engine_cost(pl, B, M, R, Tout, K);
    if (flip) return run + 4.0 + 0.73 * w;
    return run + 4.9 + 0.43 * w + (Tin % 8 != 0 ? 1.0 + 2.4e-6 * B * R * Tin : 0.0);
}
// The same for a forward call on the engine for few tiles, fitted to 3248 calls that the estimates above send to unpacked
// weights, timed on both (rms 8 %): in one part that engine has no second launch.
double packed_split_device(const SplitPlan &sp, int B, int M, int R, int Tin, int K)
{
    const double w = 2e-6 * M * R * K, odd = Tin % 8 != 0 ? 1.0 : 0.0;
    if (sp.nsplit == 1) return 7.5 + 0.81 * sp.device + 0.66 * w + 1.6 * odd;
    return 13.0 + 0.71 * sp.device + 0.31 * w + odd * 1.1e-6 * B * R * Tin;
}
// The plan on unpacked weights where it is the better one by more than the estimates err (over those 345).  Against the engine
// for few tiles also with three parts at least (in two it lost in 37 of 66 calls), and in forward calls by that later fit
// too: 128 -> 1024 channels, K=11, B=10, T=203 20.3 us packed, 31.1 unpacked; 256 -> 512, K=13, B=23, T=203 34 / 47.  187
// calls that these two keep packed: 8 % faster so on average, 12 of them slower by more than 4 %.
UnpackedPlan better_unpacked(const Plan &pl, const SplitPlan &sp, int B, int M, int R, int Tin, int Tout, int K, int dil, bool flip, size_t part_limit)
{
    if (!pl.ok || !unpacked_supported(M, R, K, pl.stride, flip)) return UnpackedPlan{};
    const double most = 0.92 * packed_cost(pl, sp, B, M, R, Tin, Tout, K, flip);
    // (whatever the plan, its multiplications spread evenly: most large calls need not be looked at any further)
    if (10.7 + 0.69 * 0.0444 / 4 / 256 * ((M + kTileM - 1) / kTileM) * (R / 16) * (double)B * ((Tout + 31) / 32) * K > most) return UnpackedPlan{};
    const UnpackedPlan up = unpacked_plan(B, M, R, Tout, K, dil, flip, part_limit);
    if (!up.nt || up.cost >= most || (sp.nt && up.nsplit < 3)) return UnpackedPlan{};
    return flip || !sp.nt || up.device < packed_split_device(sp, B, M, R, Tin, K) ? up : UnpackedPlan{};
}

size_t packed_bytes(int M, int R, int K)
{
    const size_t nmt = (M + kTileM - 1) / kTileM, nch = (R + kChunk - 1) / kChunk;
    const size_t Kp = (size_t)((K + 1) & ~1);
    return align_up((nmt * nch * Kp * 256 + 512) * sizeof(u32x4), 256);  // + one tap pair of zeros
}

constexpr size_t kMaxPacked = (size_t)1 << 31;  // the kernel addresses packed weights with 32-bit offsets
constexpr size_t kMaxInput = (size_t)1 << 30;   // and the activation tensors through buffer descriptors

template <int NT, int STRIDE, int KT, bool LEN = false, bool STATS = false, bool ANYROW = false, bool PADPAIR = false>
hipError_t launch_t(const ConvGemmParams &p, size_t lds, hipStream_t s)
{
    auto kern = conv_gemm_kernel<NT, STRIDE, KT, LEN, STATS, ANYROW, PADPAIR>;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), kMaxLds);
    if (e != hipSuccess) return e;
    const int cus = current_device_info().cus;
    const int grid = p.num_tiles < cus ? p.num_tiles : cus;
    ConvGemmParams q = p;
    // private tiles per wavefront (unrolled kernels only); a remainder of more than two shared rounds
    // is cheaper as one more private round in which some wavefronts stay idle: no exchange epilogues, and
    // on a chip that runs at its power limit the idle wavefronts' share of the budget raises the clock of
    // the busy ones (256 channels, K=11, B=32: 640 tiles on 1024 wavefronts, step 173 -> 159 us)
    q.full = KT > 0 ? p.num_tiles / (kWaves * grid) + (p.num_tiles % (kWaves * grid) > 2 * grid ? 1 : 0) : 0;
    MainKernelTimer timer(s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, q);
    return hipGetLastError();
}

template <bool LEN, int MI, int NT, int SC>
hipError_t launch_pointwise_shape(const ConvGemmParams &p, hipStream_t s)
{
    using Sh = PwShape<MI, NT, SC>;
    auto kern = pointwise_gemm_kernel<LEN, MI, NT, SC>;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), (int)Sh::kLds);
    if (e != hipSuccess) return e;
    ConvGemmParams q = p;
    q.ntt = (p.Tout + NT * 32 - 1) / (NT * 32);
    const int cus = current_device_info().cus;
    const int ntiles = (p.nmt + kWaves * Sh::kRowTiles - 1) / (kWaves * Sh::kRowTiles) * q.ntt * p.B;
    MainKernelTimer timer(s);
    hipLaunchKernelGGL(kern, dim3(ntiles < cus ? ntiles : cus), dim3(kThreads), Sh::kLds, s, q);
    return hipGetLastError();
}

hipError_t launch_pointwise(const ConvGemmParams &p, bool big, bool len, hipStream_t s)
{
    if (len)
        return big ? launch_pointwise_shape<true, 4, 4, 64>(p, s) : launch_pointwise_shape<true, 2, 5, 128>(p, s);
    return big ? launch_pointwise_shape<false, 4, 4, 64>(p, s) : launch_pointwise_shape<false, 2, 5, 128>(p, s);
}

hipError_t launch_few_channels(const ConvGemmParams &p, hipStream_t s)
{
    const int nstrips = (p.Tout + kFewStrip - 1) / kFewStrip;
    MainKernelTimer timer(s);
    // the output channels of a strip are shared out among the workgroups of a column of the grid: enough
    // workgroups to give every SIMD several wavefronts (the stores are the work)
    const int cus = current_device_info().cus;
    const int nblocks = (p.M + 31) / 32;
    int split = 1;
    while (split < 8 && p.B * nstrips * split < 4 * cus && nblocks >= 2 * kWaves * split) split *= 2;
    hipLaunchKernelGGL(few_channels_gemm_kernel, dim3(p.B * nstrips, split), dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

template <int NT, int STRIDE>
hipError_t launch_split_t(ConvGemmParams p, int cols_at_once, size_t lds, hipStream_t s, SplitSum *later)
{
    MainKernelTimer timer(s);
    const int cols = p.ntt * p.B;
    for (p.col0 = 0; p.col0 < cols; p.col0 += cols_at_once) {
        p.ncols = std::min(cols_at_once, cols - p.col0);
        hipLaunchKernelGGL((conv_split_kernel<NT, STRIDE>), dim3(p.nmt * p.ncols * p.nsplit), dim3(kThreads), lds, s, p);
        const hipError_t e = p.nsplit > 1 ? launch_split_reduce(p, NT, s, cols_at_once >= cols && !timer.stop ? later : nullptr) : hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// [part, part + part_room): room for the parts of one column of tiles at least
hipError_t launch_split(const SplitPlan &sp, const ConvGemmParams &p0, int stride, void *part, size_t part_room, hipStream_t s, SplitSum *later)
{
    ConvGemmParams p = p0;
    p.ntt = (p.Tout + sp.nt * 32 - 1) / (sp.nt * 32);
    p.num_tiles = p.nmt * p.ntt * p.B;
    p.nsplit = sp.nsplit;
    p.nitems = sp.ngroups;
    p.buf_bytes = sp.ngroups * 8 * kRowBytes;
    p.part = (f32x4 *)part;
    const int cols = p.ntt * p.B;
    const int at_once = sp.part_bytes <= part_room ? cols : (int)(part_room / sp.col_bytes);
    if (at_once < 1) return hipErrorInvalidValue;  // (no such plan is made)
    if (stride == 1) {
        if (sp.nt == 4) return launch_split_t<4, 1>(p, at_once, sp.lds, s, later);
        if (sp.nt == 3) return launch_split_t<3, 1>(p, at_once, sp.lds, s, later);
        return launch_split_t<2, 1>(p, at_once, sp.lds, s, later);
    }
    if (sp.nt == 3) return launch_split_t<3, 2>(p, at_once, sp.lds, s, later);
    return launch_split_t<2, 2>(p, at_once, sp.lds, s, later);
}

// Calls of conv_rows_kernel: those that have an instance (stride 2, K = 11; the six taps of its gradient, two row tiles) and enough
// workgroups.  In a sweep over 32 to 256 input and 192 to 512 output channels, 50 to 51200 steps, the lines below
// separate gains (forward 1.1 to 1.5 times, gradient up to 1.5) from losses but for a few per cent: forward 64 -> 256, B=24,
// T=1000, 192 workgroups 15.2 us on conv_split_kernel, 15.6 here; B=20, T=1203, 200 of them 23.2 / 17.6; gradient, 64
// workgroups 24.8 / 24.9, 84 29.4 / 28.2.  The wavefronts of a row group that is
// half full or less wait for the others, which costs most where a last round of workgroups is nearly empty: 600 calls of up to 1024 input
// channels take 0.85 of the time on average, the worst 1.06, where that goes to the engine for few tiles (638 -> 384, B=28, T=528, 24 workgroups
// in the last round, 60.0 us there, 91.5 here; 118 -> 300, B=24, T=1352, 16 of them, 39.1 / 45.8; 273 -> 257, B=24, T=800, 80 of them
// 53.6 / 48.8).  Layers of six taps and stride 1 run the gradient's instance; with few chunks it needs more workgroups for its longer start (50
// channels and 90 workgroups 11.5 / 13.0, 96 and 138 13.3 / 14.7, 50 and 387 20.4 / 19.2).
// (phases: both parities of a strided gradient)
bool takes_rows(const Plan &pl, const SplitPlan &sp, int B, int M, int R, int Tout, int K, int dil, bool phases)
{
    const int nmt = (M + kTileM - 1) / kTileM;
    if (!pl.ok || dil != 1) return false;
    if (pl.stride == 2) {
        const long cols = (long)B * ((Tout + 63) / 64), wgs = cols * ((nmt + 3) / 4);
        const bool idle = (nmt & 3) == 1 || (nmt & 3) == 2, thin = wgs > 256 && wgs % 256 > 0 && wgs % 256 <= 96;
        return K == 11 && nmt >= 3 && cols * nmt >= 4 * 200 && !(sp.nt && idle && thin);
    }
    const int least = phases ? 80 : std::max(80, 256 - 32 * ((R + kChunk - 1) / kChunk));
    return K == 6 && nmt == 2 && M >= 96 && (long)B * ((Tout + 127) / 128) >= least;  // (a second tile that is at least half full)
}
template <int STRIDE, int WM, int KT>
hipError_t launch_rows_t(ConvGemmParams p, hipStream_t s)
{
    using Sh = RowsShape<STRIDE, WM, KT>;
    static_assert(Sh::LDS <= 64 * 1024, "LDS without an opt-in");
    p.ntt = (p.Tout + Sh::COLS - 1) / Sh::COLS;
    MainKernelTimer timer(s);
    hipLaunchKernelGGL((conv_rows_kernel<STRIDE, WM, KT>), dim3((unsigned)((p.nmt + WM - 1) / WM * p.ntt * p.B)), dim3(kThreads), Sh::LDS, s, p);
    return hipGetLastError();
}

// Which kernel makes a contraction.
struct ConvChoice {
    enum Kind { kFew, kSplit, kPointwise, kRows, kGemm } kind;
    bool big;                                // kPointwise: the 512 x 128 tile
    int nt, stride, kt;                      // kGemm: the template arguments (stride: of kRows too)
    bool len, stats, any, pad_pair;          // (len: of kPointwise too)
};
ConvChoice choose_conv(const Plan &pl, const SplitPlan &sp, const ConvGemmParams &p)
{
    ConvChoice c = {};
    c.any = p.odd_rows != 0;
    // one tap, at most one chunk of reduction channels, nothing to do after the sums: the store-bound kernel
    if (p.K == 1 && p.R <= kChunk && pl.stride == 1 && p.padL == 0 && p.Tin == p.Tout && p.Tout % 8 == 0 && !p.res &&
        !p.scale && !p.shift && !p.relu && !p.len_in && !p.len_out) {
        c.kind = ConvChoice::kFew;
        return c;
    }
    if (!p.stats && takes_rows(pl, sp, p.B, p.M, p.R, p.Tout, p.K, p.dil, p.len_out_div == 2)) {
        c.kind = ConvChoice::kRows;
        c.stride = pl.stride;
        return c;
    }
    if (!p.stats && sp.nt) {
        c.kind = ConvChoice::kSplit;
        return c;
    }
    // one tap, no padding, wide tiles: the GEMM kernel whose wavefronts share the staged activations
    // (worth it from two 64-channel row tiles on: a single one would leave three wavefronts idle)
    if (p.K == 1 && p.nmt >= 2 && pl.nt == 5 && pl.stride == 1 && p.padL == 0 && p.Tin == row_pitch(p.Tout)) {
        c.kind = ConvChoice::kPointwise;
        c.big = pointwise_big_tile(p, current_device_info().cus);
        c.len = p.len_in || c.any;
        return c;
    }
    c.kind = ConvChoice::kGemm;
    c.nt = pl.nt;
    c.stride = pl.stride;
    c.stats = p.stats != nullptr;  // (the caller has checked that the unrolled kernel serves the call)
    c.kt = pl.unrolled || c.stats ? p.K : 0;
    c.len = c.kt > 0 && (c.any || p.len_in || p.len_out) && !c.stats;
    // (a wavefront has an odd number of pairs where both a chunk's pairs and its chunks are odd)
    c.pad_pair = c.any && c.kt == 0 && p.Kp / 2 % 2 && p.nch % (2 * kWaves) != 0;
    return c;
}

template <bool LEN, bool STATS, bool ANY>
hipError_t launch_unrolled(int kt, const ConvGemmParams &p, size_t lds, hipStream_t s)
{
    switch (kt) {
    case 11: return launch_t<5, 1, 11, LEN, STATS, ANY>(p, lds, s);
    case 13: return launch_t<5, 1, 13, LEN, STATS, ANY>(p, lds, s);
    case 17: return launch_t<5, 1, 17, LEN, STATS, ANY>(p, lds, s);
    case 21: return launch_t<5, 1, 21, LEN, STATS, ANY>(p, lds, s);
    case 25: return launch_t<5, 1, 25, LEN, STATS, ANY>(p, lds, s);
    case 29: return launch_t<5, 1, 29, LEN, STATS, ANY>(p, lds, s);
    default: return hipErrorInvalidValue;
    }
}
template <bool ANY, bool PAD>
hipError_t launch_tap_pairs(const ConvChoice &c, const ConvGemmParams &p, size_t lds, hipStream_t s)
{
    if (c.nt == 5 && c.stride == 1) return launch_t<5, 1, 0, false, false, ANY, PAD>(p, lds, s);
    if (c.nt == 2 && c.stride == 1) return launch_t<2, 1, 0, false, false, ANY, PAD>(p, lds, s);
    if (c.nt == 2 && c.stride == 2) return launch_t<2, 2, 0, false, false, ANY, PAD>(p, lds, s);
    return hipErrorInvalidValue;
}

// [part, part + part_room): room for the partial sums of the split engine, whose plan is sp
hipError_t launch_plan(const Plan &pl, const SplitPlan &sp, const ConvGemmParams &p, hipStream_t s, void *part, size_t part_room,
                       SplitSum *later = nullptr)
{
    const ConvChoice c = choose_conv(pl, sp, p);
    switch (c.kind) {
    case ConvChoice::kFew: return launch_few_channels(p, s);
    case ConvChoice::kSplit: return launch_split(sp, p, pl.stride, part, part_room, s, later);
    case ConvChoice::kPointwise: return launch_pointwise(p, c.big, c.len, s);
    case ConvChoice::kRows: return c.stride == 2 ? launch_rows_t<2, 4, 11>(p, s) : launch_rows_t<1, 2, 6>(p, s);
    case ConvChoice::kGemm: break;
    }
    if (c.stats) return launch_unrolled<false, true, false>(c.kt, p, pl.lds, s);
    if (c.kt > 0)
        return c.any ? launch_unrolled<true, false, true>(c.kt, p, pl.lds, s)
                     : c.len ? launch_unrolled<true, false, false>(c.kt, p, pl.lds, s) : launch_unrolled<false, false, false>(c.kt, p, pl.lds, s);
    if (c.any) return c.pad_pair ? launch_tap_pairs<true, true>(c, p, pl.lds, s) : launch_tap_pairs<true, false>(c, p, pl.lds, s);
    return launch_tap_pairs<false, false>(c, p, pl.lds, s);
}

// the kernel's name as a profiler lists it
void name_conv(const Plan &pl, const SplitPlan &sp, const ConvGemmParams &p, char *name, size_t n)
{
    const ConvChoice c = choose_conv(pl, sp, p);
    auto b = [](bool v) { return v ? "true" : "false"; };
    switch (c.kind) {
    case ConvChoice::kFew: snprintf(name, n, "few_channels_gemm_kernel"); break;
    case ConvChoice::kSplit: snprintf(name, n, "conv_split_kernel<%d, %d> in %d parts", sp.nt, pl.stride, sp.nsplit); break;
    case ConvChoice::kPointwise:
        snprintf(name, n, "pointwise_gemm_kernel<%s, %s>", b(c.len), c.big ? "4, 4, 64" : "2, 5, 128");
        break;
    case ConvChoice::kRows: snprintf(name, n, "conv_rows_kernel<%s>", c.stride == 1 ? "1, 2, 6" : "2, 4, 11"); break;
    case ConvChoice::kGemm:
        snprintf(name, n, "conv_gemm_kernel<%d, %d, %d, %s, %s, %s, %s>", c.nt, c.stride, c.kt, b(c.len), b(c.stats), b(c.any), b(c.pad_pair));
        break;
    }
}

size_t prepack_lds(int K) { return (size_t)kPackRows * pack_m_stride(K) * sizeof(bf16_t); }

// flip == false: W'[m][r][k] = w[m][r][k] (w is [M][R][K]); flip == true: W'[m][r][k] = w[r][m][K-1-k] * rscale[r]
// (w is [R][M][K]; rscale NULL: 1).
struct PackGeom {
    int nmt, nch, vec;
    size_t lds, zero_off;
    unsigned blocks;
};
PackGeom pack_geom(const void *w, int M, int R, int K, bool flip)
{
    PackGeom q;
    q.nmt = (M + kTileM - 1) / kTileM;
    q.nch = (R + kChunk - 1) / kChunk;
    q.lds = prepack_lds(K);
    q.zero_off = (size_t)q.nmt * q.nch * ((K + 1) & ~1) * 256;
    // runs start at multiples of 2*K*(row length) bytes from w: 16-byte aligned when w is and the other
    // channel count is a multiple of 8 (the tensor must also fit a 32-bit byte offset)
    const int other = flip ? M : R;
    q.vec = ((uintptr_t)w % 16 == 0 && other % 8 == 0 && (size_t)M * R * K * 2 < ((size_t)1 << 31)) ? 1 : 0;
    q.blocks = (unsigned)(q.nmt * q.nch * 4);
    return q;
}

hipError_t run_prepack(const void *w, void *wp, int M, int R, int K, bool flip, const float *rscale, hipStream_t s)
{
    const PackGeom q = pack_geom(w, M, R, K, flip);
    hipError_t e;
    if (flip) {
        static LdsOptIn opt_in;
        e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(prepack_kernel<true>), kMaxLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(prepack_kernel<true>, dim3(q.blocks), dim3(256), q.lds, s, (const bf16_t *)w, (u32x4 *)wp,
                           M, R, K, q.nch, M * K, q.zero_off, q.vec, rscale);
    } else {
        static LdsOptIn opt_in;
        e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(prepack_kernel<false>), kMaxLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(prepack_kernel<false>, dim3(q.blocks), dim3(256), q.lds, s, (const bf16_t *)w, (u32x4 *)wp,
                           M, R, K, q.nch, R * K, q.zero_off, q.vec, (const float *)nullptr);
    }
    return hipGetLastError();
}

}  // namespace
hipError_t launch_prepare_rows(const Geom &g, const RowPrep &r, hipStream_t s)
{
    PrepareRowsArgs a = {};
    size_t lds = 0;
    if (r.w) {
        a.M = r.flip ? g.Cin : g.Cout;
        a.R = r.flip ? g.Cout : g.Cin;
        const PackGeom q = pack_geom(r.w, a.M, a.R, g.K, r.flip);
        a.npack = q.blocks;
        a.w = (const bf16_t *)r.w;
        a.wp = (u32x4 *)r.wp;
        a.K = g.K; a.nch = q.nch; a.ld = (r.flip ? a.M : a.R) * g.K; a.vec = q.vec;
        a.zero_off = q.zero_off;
        a.rscale = r.rscale;
        lds = q.lds;
    }
    if (r.dy) {
        a.B = g.B; a.Cout = g.Cout; a.To = g.To;
        a.ncm = r.gf ? r.ncm : (g.Cout + 31) / 32;
        a.nst = r.gf ? r.nst : (g.To + 15) / 16;
        a.nst4 = (a.nst + 3) / 4;
        a.nmask = (unsigned)(((size_t)g.B * a.ncm * a.nst4 + 3) / 4);
        a.dy = (const bf16_t *)r.dy;
        a.y = (const bf16_t *)r.y;
        a.relu = r.relu ? 1 : 0;
        a.gplain = (bf16_t *)r.gplain;
        a.dres = (bf16_t *)r.dres;
        a.gf = (u32x4 *)r.gf;
    }
    unsigned ncopy = 0;
    if (r.x) {
        a.Cin = g.Cin; a.T = g.T; a.T8 = row_pitch(g.T) / 8;
        a.ngroups = (size_t)g.B * g.Cin * a.T8;
        a.len = g.len;
        a.x = (const bf16_t *)r.x;
        a.xp = (u32x4 *)r.xp;
        ncopy = (unsigned)((a.ngroups + 255) / 256);
    }
    const unsigned blocks = a.npack + a.nmask + ncopy;
    if (blocks == 0) return hipSuccess;
    hipError_t e;
    if (r.flip) {
        static LdsOptIn opt_in;
        e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(prepare_rows_kernel<true>), kMaxLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(prepare_rows_kernel<true>, dim3(blocks), dim3(256), lds, s, a);
    } else {
        static LdsOptIn opt_in;
        e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(prepare_rows_kernel<false>), kMaxLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(prepare_rows_kernel<false>, dim3(blocks), dim3(256), lds, s, a);
    }
    return hipGetLastError();
}
namespace {

void fill_common(ConvGemmParams &p, const Plan &pl, int B, int M, int R, int Tin, int Tout, int K, int dil, int padL, bool odd_rows)
{
    p.odd_rows = odd_rows ? 1 : 0;
    p.B = B; p.M = M; p.R = R; p.Tin = Tin; p.Tout = Tout; p.K = K; p.Kp = (K + 1) & ~1; p.dil = dil; p.padL = padL;
    p.nmt = (M + kTileM - 1) / kTileM;
    p.nch = (R + kChunk - 1) / kChunk;
    p.ntt = (Tout + pl.nt * 32 - 1) / (pl.nt * 32);
    p.num_tiles = p.nmt * p.ntt * B;
    p.wp_zero = (size_t)p.nmt * p.nch * p.Kp * 256;
    p.wp_bytes = (p.wp_zero + 512) * sizeof(u32x4);
    p.nitems = pl.nitems;
    p.buf_bytes = pl.buf_bytes;
    p.overlap = pl.overlap;
}

}  // namespace

// (also reports a refused launch before it: asking clears it)
hipError_t launch_split_reduce(const ConvGemmParams &p, int nt, hipStream_t s, SplitSum *later)
{
    if (later) {
        later->set = true;
        later->p = p;
        later->nt = nt;
        return hipGetLastError();
    }
    hipLaunchKernelGGL(split_reduce_kernel, dim3(p.nmt * p.ncols * kWaves * nt), dim3(64), 0, s, p, nt);
    return hipGetLastError();
}

// ---- forward ---------------------------------------------------------------------------
bool mfma_fwd_supported(const Geom &g)
{
    if ((size_t)g.B * g.Cin * row_pitch(g.T) * sizeof(bf16_t) > kMaxInput) return false;
    if ((size_t)g.B * g.Cout * row_pitch(g.To) * sizeof(bf16_t) > kMaxInput) return false;
    return packed_bytes(g.Cout, g.Cin, g.K) < kMaxPacked && make_plan(row_pitch(g.T), g.To, g.Cin, g.K, g.stride, g.dil).ok;
}

size_t mfma_fwd_workspace_least(const Geom &g) { return packed_bytes(g.Cout, g.Cin, g.K) + pitched_x_bytes(g); }
namespace {
// Where the best plan's parts do not fit: a plan in fewer, else another engine (a plan in one part is close to that, and the
// estimates are not close enough to tell: 896 -> 16 channels, K=29, B=2, T=304 83 us in one part, 75 there).
SplitPlan in_parts(const SplitPlan &sp) { return sp.nsplit > 1 ? sp : SplitPlan{}; }
// the plan with ws_bytes of workspace; in_rounds: that of a call with the workspace it asks for, whatever the room
SplitPlan fwd_split_plan(const Geom &g, const Plan &pl, size_t ws_bytes, bool in_rounds = false)
{
    const size_t least = mfma_fwd_workspace_least(g), room = ws_bytes > least ? ws_bytes - least : 0;
    const bool array = least <= NM_STATIC_SCRATCH_BYTES;
    const SplitPlan sp = split_plan(pl, g.B, g.Cout, g.Cin, g.To, g.K, g.dil, array ? NM_STATIC_SCRATCH_BYTES - least : kNoLimit, kSplitRounds);
    return sp.part_bytes <= room || in_rounds ? sp : in_parts(split_plan(pl, g.B, g.Cout, g.Cin, g.To, g.K, g.dil, room));
}
// The same on unpacked weights.  The parts lie behind the room of a call on packed ones; nm_conv1d_block_fwd_static, whose
// array has that room free, keeps them there, so the plan of a call it serves has parts of that size at most.
UnpackedPlan fwd_unpacked_plan(const Geom &g, const Plan &pl, size_t ws_bytes, bool in_rounds = false)
{
    const size_t least = mfma_fwd_workspace_least(g), room = ws_bytes > least ? ws_bytes - least : 0;
    const SplitPlan sp = fwd_split_plan(g, pl, ws_bytes, in_rounds);
    auto plan = [&](size_t limit) { return better_unpacked(pl, sp, g.B, g.Cout, g.Cin, g.T, g.To, g.K, g.dil, false, limit); };
    const UnpackedPlan up = plan(least <= NM_STATIC_SCRATCH_BYTES ? NM_STATIC_SCRATCH_BYTES : kNoLimit);
    return up.part_bytes <= room || in_rounds ? up : plan(room);
}
}  // namespace
size_t mfma_fwd_workspace(const Geom &g)
{
    const Plan pl = make_plan(row_pitch(g.T), g.To, g.Cin, g.K, g.stride, g.dil);
    return mfma_fwd_workspace_least(g) + std::max(fwd_split_plan(g, pl, kNoLimit).part_bytes, fwd_unpacked_plan(g, pl, kNoLimit).part_bytes);
}

// Whether the forward pass of this geometry runs on a kernel instance that can also write the statistics of its
// outputs, and into how many (batch item, time tile) parts: the unrolled engine, wide tile, no lengths, 16-byte rows.
int mfma_fwd_stats_parts(const Geom &g, const void *w, size_t ws_bytes)
{
    if (!rows16(g)) return 0;
    const Plan pl = make_plan(g.T, g.To, g.Cin, g.K, g.stride, g.dil);
    if (!pl.ok || !pl.unrolled || pl.nt != 5 || g.len || !mfma_fwd_supported(g)) return 0;
    if (pl.buf_bytes < Epilogue<5>::kTileBytesWithStats) return 0;
    // few tiles: z is small and read again instead, where the engine for those saves more than that takes
    const SplitPlan sp = fwd_split_plan(g, pl, ws_bytes);
    if (sp.nt && sp.gain > 3.0) return 0;
    const UnpackedPlan up = ((uintptr_t)w % 16) == 0 ? fwd_unpacked_plan(g, pl, ws_bytes) : UnpackedPlan{};
    if (up.nt && packed_cost(pl, SplitPlan{}, g.B, g.Cout, g.Cin, g.T, g.To, g.K, false) - up.cost > 5.0) return 0;
    return g.B * ((g.To + 159) / 160);
}

hipError_t launch_mfma_fwd(const Geom &g, const void *x, const void *w, const float *scale, const float *shift,
                           const void *res, void *y, bool relu, void *ws, size_t ws_bytes, hipStream_t s, double *stats, bool in_rounds)
{
    const Plan pl = make_plan(row_pitch(g.T), g.To, g.Cin, g.K, g.stride, g.dil);
    if (!pl.ok || !mfma_fwd_supported(g)) return hipErrorInvalidValue;
    if (stats && mfma_fwd_stats_parts(g, w, ws_bytes) == 0) return hipErrorInvalidValue;
    // a pointwise layer with a handful of output channels is a stream over x: no packing, no tiles
    if (skinny_fwd_supported(g) && ((uintptr_t)w % 16) == 0) return launch_skinny_fwd(g, x, w, scale, shift, res, y, relu, s);
    hipError_t e;
    const void *in = x;
    const size_t least = mfma_fwd_workspace_least(g);
    auto fill = [&](ConvGemmParams &p, int Tin) {
        fill_common(p, pl, g.B, g.Cout, g.Cin, Tin, g.To, g.K, g.dil, g.pad, !rows16(g));
        p.relu = relu ? 1 : 0;
        p.in = (const bf16_t *)in;
        p.len_in = g.len;
        p.wp = (const bf16x8 *)ws;
        p.scale = scale; p.shift = shift; p.res = (const bf16_t *)res;
        p.out = (bf16_t *)y;
        p.stats = stats;
    };
    if (!stats && ((uintptr_t)w % 16) == 0) {
        const UnpackedPlan up = fwd_unpacked_plan(g, pl, ws_bytes, in_rounds);
        if (up.nt) {
            ConvGemmParams p = {};
            fill(p, g.T);
            return launch_unpacked_conv(up, p, w, false, nullptr, (unsigned char *)ws + (in_rounds ? 0 : least), s);
        }
    }
    if (g.T % 8 == 0) {
        e = run_prepack(w, ws, g.Cout, g.Cin, g.K, false, nullptr, s);
    } else {
        RowPrep a = {};
        a.w = w;
        a.wp = ws;
        a.x = x;
        a.xp = (unsigned char *)ws + packed_bytes(g.Cout, g.Cin, g.K);
        in = a.xp;
        e = launch_prepare_rows(g, a, s);
    }
    if (e != hipSuccess) return e;
    ConvGemmParams p = {};
    fill(p, row_pitch(g.T));
    return launch_plan(pl, fwd_split_plan(g, pl, ws_bytes, in_rounds), p, s, (unsigned char *)ws + least, ws_bytes > least ? ws_bytes - least : 0);
}

namespace {
void name_unpacked(const UnpackedPlan &up, int K, bool flip, char *name, size_t n)
{
    snprintf(name, n, "conv_unpacked_kernel<%d, %d, %s> in %d parts", up.nt, K, flip ? "true" : "false", up.nsplit);
}
}  // namespace
void name_mfma_fwd(const Geom &g, bool stats, size_t ws_bytes, char *name, size_t n)
{
    if (skinny_fwd_supported(g)) {
        snprintf(name, n, "decoder_mfma_kernel<true, %s, %d>", g.T % 8 == 0 ? "false" : "true", decoder_split(g.B, g.Cin, g.T));
        return;
    }
    static float affine;
    static double some_stats;
    const Plan pl = make_plan(row_pitch(g.T), g.To, g.Cin, g.K, g.stride, g.dil);
    ConvGemmParams p = {};
    fill_common(p, pl, g.B, g.Cout, g.Cin, row_pitch(g.T), g.To, g.K, g.dil, g.pad, !rows16(g));
    p.len_in = g.len;
    p.scale = &affine;
    if (stats && mfma_fwd_stats_parts(g, nullptr, ws_bytes) > 0) p.stats = &some_stats;
    const UnpackedPlan up = p.stats ? UnpackedPlan{} : fwd_unpacked_plan(g, pl, ws_bytes);
    if (up.nt) return name_unpacked(up, g.K, false, name, n);
    name_conv(pl, fwd_split_plan(g, pl, ws_bytes), p, name, n);
}

// ---- input gradient (stride 1 only; other strides use the plain kernels) ----------------
// Workspace: packed (flipped, transposed) weights, then dz when it differs from dy.
namespace {
// (16-byte rows of T % 16 == 8 keep the plain kernel, whose smaller workspace they were always served with)
Phases phases_of_stride2(const Geom &g)
{
    Phases ph = {};
    if (g.stride != 2 || g.dil != 1 || (rows16(g) && g.T % 16 != 0)) return ph;
    int padL[2];
    for (int r = 0; r < 2; ++r) {
        ph.kp[r] = (r + g.pad) & 1;
        ph.Kr[r] = g.K > ph.kp[r] ? (g.K - ph.kp[r] + 1) / 2 : 0;
        if (ph.Kr[r] < 1) return ph;
        // out[u] = sum_j W'[j] * g[u - padL + j] with j = Kr-1-k'
        padL[r] = ph.Kr[r] - 1 - (r + g.pad - ph.kp[r]) / 2;
    }
    ph.padL = std::max(padL[0], padL[1]);
    for (int r = 0; r < 2; ++r) ph.K = std::max(ph.K, ph.Kr[r] + ph.padL - padL[r]);
    for (int r = 0; r < 2; ++r) ph.off[r] = ph.K - ph.Kr[r] - (ph.padL - padL[r]);
    ph.U = (g.T + 1) / 2;
    ph.Up = row_pitch(ph.U);
    ph.ok = make_plan(row_pitch(g.To), ph.Up, g.Cout, ph.K, 1, 1).ok && packed_bytes(2 * g.Cin, g.Cout, ph.K) < kMaxPacked &&
            (size_t)g.B * 2 * g.Cin * ph.Up * sizeof(bf16_t) <= kMaxInput;
    return ph;
}
size_t phase_bytes(const Geom &g, const Phases &ph)  // the parities' outputs
{
    return align_up((size_t)g.B * 2 * g.Cin * ph.Up * sizeof(bf16_t), 256);
}
size_t dz_bytes_of(const Geom &g) { return align_up((size_t)g.B * g.Cout * row_pitch(g.To) * sizeof(bf16_t), 256); }
}  // namespace

bool mfma_dgrad_supported(const Geom &g)
{
    if ((size_t)g.B * g.Cout * row_pitch(g.To) * sizeof(bf16_t) > kMaxInput) return false;
    if ((size_t)g.B * g.Cin * row_pitch(g.T) * sizeof(bf16_t) > kMaxInput) return false;
    if (g.stride == 2) return phases_of_stride2(g).ok;
    if (g.stride != 1 || packed_bytes(g.Cin, g.Cout, g.K) >= kMaxPacked) return false;
    return make_plan(row_pitch(g.To), g.T, g.Cout, g.K, 1, g.dil).ok;
}

size_t mfma_dgrad_workspace_least(const Geom &g)
{
    if (g.stride == 2) {
        const Phases ph = phases_of_stride2(g);
        return dz_bytes_of(g) + packed_bytes(2 * g.Cin, g.Cout, ph.K) + phase_bytes(g, ph);
    }
    return packed_bytes(g.Cin, g.Cout, g.K) + dz_bytes_of(g);
}
namespace {
SplitPlan dgrad_split_plan(const Geom &g, const Plan &pl, size_t ws_bytes)
{
    const size_t least = mfma_dgrad_workspace_least(g), room = ws_bytes > least ? ws_bytes - least : 0;
    const Phases ph = g.stride == 2 ? phases_of_stride2(g) : Phases{};
    auto plan = [&](size_t limit) {
        return g.stride == 2 ? split_plan(pl, g.B, 2 * g.Cin, g.Cout, ph.Up, ph.K, 1, limit)
                             : split_plan(pl, g.B, g.Cin, g.Cout, g.T, g.K, g.dil, limit);
    };
    const SplitPlan sp = plan(kNoLimit);
    return sp.part_bytes <= room ? sp : in_parts(plan(room));
}
UnpackedPlan dgrad_unpacked_plan(const Geom &g, const Plan &pl, size_t ws_bytes)
{
    if (g.stride != 1) return UnpackedPlan{};
    const size_t least = mfma_dgrad_workspace_least(g), room = ws_bytes > least ? ws_bytes - least : 0;
    const SplitPlan sp = dgrad_split_plan(g, pl, ws_bytes);
    auto plan = [&](size_t limit) { return better_unpacked(pl, sp, g.B, g.Cin, g.Cout, row_pitch(g.To), g.T, g.K, g.dil, true, limit); };
    const UnpackedPlan up = plan(kNoLimit);
    return up.part_bytes <= room ? up : plan(room);
}
}  // namespace
bool mfma_dgrad_unpacked(const Geom &g, const void *w, size_t ws_bytes)
{
    return g.stride == 1 && ((uintptr_t)w % 16) == 0 &&
           dgrad_unpacked_plan(g, make_plan(row_pitch(g.To), g.T, g.Cout, g.K, 1, g.dil), ws_bytes).nt != 0;
}
size_t mfma_dgrad_workspace(const Geom &g)
{
    const Phases ph = g.stride == 2 ? phases_of_stride2(g) : Phases{};
    const Plan pl = g.stride == 2 ? make_plan(row_pitch(g.To), ph.Up, g.Cout, ph.K, 1, 1) : make_plan(row_pitch(g.To), g.T, g.Cout, g.K, 1, g.dil);
    return mfma_dgrad_workspace_least(g) + std::max(dgrad_split_plan(g, pl, kNoLimit).part_bytes, dgrad_unpacked_plan(g, pl, kNoLimit).part_bytes);
}

namespace {
// The elementwise pass in front of an input gradient whose weights are packed separately: g = dy*[y>0]
// into `gbuf` (when there is a ReLU) and/or `dres`.  Returns the tensor the engine contracts in *g_used.
hipError_t mask_pass(const Geom &g, const void *dy, const void *y, bool relu, void *gbuf, void *dres, const void **g_used,
                     hipStream_t s)
{
    *g_used = dy;
    if (!relu && !dres) return hipSuccess;
    hipError_t e;
    if (dres && ((uintptr_t)dres % 16) == 0) {
        // the residual gradient is g itself: write it once and contract it from there
        e = launch_epilogue_bwd_vec8(g, dy, y, nullptr, relu, nullptr, dres, s);
        if (relu) *g_used = dres;
    } else if (!dres) {
        e = launch_epilogue_bwd_vec8(g, dy, y, nullptr, relu, gbuf, nullptr, s);
        *g_used = gbuf;
    } else {  // a misaligned dres: the 2-byte kernel writes it and an aligned copy for the engine
        e = launch_epilogue_bwd(g, true, dy, y, nullptr, relu, relu ? gbuf : nullptr, dres, s);
        if (relu) *g_used = gbuf;
    }
    return e;
}

hipError_t launch_mfma_dgrad_stride2(const Geom &g, const void *dy, const void *y, const float *scale, const void *w,
                                     void *dx, void *dres, bool relu, void *ws, void *part, size_t part_room, hipStream_t s,
                                     const void **g_used)
{
    const Phases ph = phases_of_stride2(g);
    if (!ph.ok) return hipErrorInvalidValue;
    unsigned char *cur = (unsigned char *)ws;
    void *gbuf = cur;
    cur += dz_bytes_of(g);
    void *packed = cur;
    cur += packed_bytes(2 * g.Cin, g.Cout, ph.K);
    bf16_t *phase_out = (bf16_t *)cur;
    // g is formed where it differs from dy in values or pitch: in dres where that is wanted and can be read 16 bytes at a time
    PrepareRowsArgs a = {};
    const bool in_dres = dres && g.To % 8 == 0 && ((uintptr_t)dres % 16) == 0;
    const bool form = relu || g.To % 8 != 0;
    const void *gin = !form ? dy : in_dres ? dres : gbuf;
    if (form || dres) {
        a.B = g.B; a.Cout = g.Cout; a.To = g.To;
        a.ncm = (g.Cout + 31) / 32;
        a.nst = (g.To + 15) / 16;
        a.nst4 = (a.nst + 3) / 4;
        a.nmask = (unsigned)(((size_t)g.B * a.ncm * a.nst4 + 3) / 4);
        a.dy = (const bf16_t *)dy;
        a.y = (const bf16_t *)y;
        a.relu = relu ? 1 : 0;
        a.gplain = form && !in_dres ? (bf16_t *)gbuf : nullptr;
        a.dres = (bf16_t *)dres;
    }
    if (g_used) *g_used = gin;
    const PackGeom q = pack_geom(w, 2 * g.Cin, g.Cout, ph.K, true);
    a.npack = q.blocks;
    a.w = (const bf16_t *)w;
    a.wp = (u32x4 *)packed;
    a.M = 2 * g.Cin; a.R = g.Cout; a.nch = q.nch; a.ld = g.K;
    a.zero_off = q.zero_off;
    a.rscale = scale;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(prepare_phases_kernel), kMaxLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(prepare_phases_kernel, dim3(a.npack + a.nmask), dim3(256), q.lds, s, a, ph);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const Plan pl = make_plan(row_pitch(g.To), ph.Up, g.Cout, ph.K, 1, 1);
    ConvGemmParams p = {};
    fill_common(p, pl, g.B, 2 * g.Cin, g.Cout, row_pitch(g.To), ph.Up, ph.K, 1, ph.padL, false);
    p.in = (const bf16_t *)gin;
    p.wp = (const bf16x8 *)packed;
    p.out = phase_out;
    p.len_out = g.len;  // both parities are padding from 2u >= len on (the merging pass clears an odd length's last one)
    p.len_out_div = 2;
    e = launch_plan(pl, dgrad_split_plan(g, pl, mfma_dgrad_workspace_least(g) + part_room), p, s, part, part_room);
    if (e != hipSuccess) return e;
    const unsigned n = (unsigned)g.B * g.Cin * ((g.T + 7) / 8);
    hipLaunchKernelGGL(interleave_phases_kernel, dim3((n + 255) / 256), dim3(256), 0, s, (const bf16_t *)phase_out, (bf16_t *)dx,
                       g.Cin, g.T, ph.Up, n, g.len, PhaseSums{g.Cout, g.To, g.K, g.pad, row_pitch(g.To), (const bf16_t *)gin, (const bf16_t *)w, scale});
    return hipGetLastError();
}

// parameters of the stride-1 input gradient as a run of the forward engine
void fill_dgrad(ConvGemmParams &p, const Plan &pl, const Geom &g, const void *gin, const void *packed, void *dx, bool accumulate)
{
    fill_common(p, pl, g.B, g.Cin, g.Cout, row_pitch(g.To), g.T, g.K, g.dil, g.dil * (g.K - 1) - g.pad, !rows16(g));
    p.relu = 0;
    p.in = (const bf16_t *)gin;
    p.wp = (const bf16x8 *)packed;
    p.out = (bf16_t *)dx;
    p.res = accumulate ? (const bf16_t *)dx : nullptr;  // dx += : every lane reads the 16 bytes it then overwrites
    p.len_out = g.len;
    p.len_out_div = 1;
}
}  // namespace

void name_mfma_dgrad(const Geom &g, bool accumulate, size_t ws_bytes, char *name, size_t n)
{
    static bf16_t dx;
    ConvGemmParams p = {};
    Plan pl;
    if (g.stride == 2) {
        const Phases ph = phases_of_stride2(g);
        pl = make_plan(row_pitch(g.To), ph.Up, g.Cout, ph.K, 1, 1);
        fill_common(p, pl, g.B, 2 * g.Cin, g.Cout, row_pitch(g.To), ph.Up, ph.K, 1, ph.padL, false);
        p.len_out = g.len;
        p.len_out_div = 2;
    } else {
        pl = make_plan(row_pitch(g.To), g.T, g.Cout, g.K, 1, g.dil);
        fill_dgrad(p, pl, g, nullptr, nullptr, &dx, accumulate);
        const UnpackedPlan up = dgrad_unpacked_plan(g, pl, ws_bytes);
        if (up.nt) return name_unpacked(up, g.K, true, name, n);
    }
    name_conv(pl, dgrad_split_plan(g, pl, ws_bytes), p, name, n);
}

// accumulate (stride 1 only): dx = bf16(dx + gradient), one rounding.
hipError_t launch_mfma_dgrad(const Geom &g, const void *dy, const void *y, const float *scale, const void *w,
                             void *dx, void *dres, bool relu, bool accumulate, void *ws, size_t ws_bytes, hipStream_t s,
                             const void **g_used, SplitSum *later)
{
    const size_t least = mfma_dgrad_workspace_least(g);
    void *part = (unsigned char *)ws + least;
    const size_t part_room = ws_bytes > least ? ws_bytes - least : 0;
    if (g_used) *g_used = nullptr;
    if (g.stride == 2) {
        if (accumulate) return hipErrorInvalidValue;
        return launch_mfma_dgrad_stride2(g, dy, y, scale, w, dx, dres, relu, ws, part, part_room, s, g_used);
    }
    const Plan pl = make_plan(row_pitch(g.To), g.T, g.Cout, g.K, 1, g.dil);
    if (!pl.ok || !mfma_dgrad_supported(g)) return hipErrorInvalidValue;
    // g = dy*[y>0] (exact in bf16) comes from one elementwise pass, which shares a launch with the weight
    // packing when it can use 16-byte accesses (To % 8 == 0 on this path; dres aligned); the affine
    // factor scale[co] is folded into the packed weights.
    hipError_t e = hipSuccess;
    const void *gin = dy;
    void *gbuf = (unsigned char *)ws + packed_bytes(g.Cin, g.Cout, g.K);
    const bool pack = !mfma_dgrad_unpacked(g, w, ws_bytes);
    if (g.To % 8 != 0) {
        const DzfLayout none = {};
        e = launch_bwd_prepare(g, dy, y, scale, w, pack, relu, ws, nullptr, none, dres, &gin, s);
        if (e != hipSuccess) return e;
    } else if (!dres || ((uintptr_t)dres % 16) == 0) {
        const int M = g.Cin, R = g.Cout;  // the engine's roles for this pass
        PackGeom q = pack_geom(w, M, R, g.K, true);
        if (!pack) q.blocks = 0, q.lds = 0;
        void *gout = dres ? dres : (relu ? gbuf : nullptr);
        const size_t n8 = gout ? (size_t)g.B * g.Cout * g.To / 8 : 0;
        const unsigned blocks = q.blocks + (unsigned)((n8 + 255) / 256);
        static LdsOptIn opt_in;
        e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(dgrad_prepare_kernel), kMaxLds);
        if (e != hipSuccess) return e;
        if (blocks)
            hipLaunchKernelGGL(dgrad_prepare_kernel, dim3(blocks), dim3(256), q.lds, s, q.blocks,
                               (const bf16_t *)w, (u32x4 *)ws, M, R, g.K, q.nch, M * g.K, q.zero_off, q.vec, scale, n8,
                               (const u32x4 *)dy, (const u32x4 *)y, relu ? 1 : 0, (u32x4 *)gout);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (relu) gin = gout;
    } else {
        if (pack) e = run_prepack(w, ws, g.Cin, g.Cout, g.K, true, scale, s);
        if (e != hipSuccess) return e;
        e = mask_pass(g, dy, y, relu, gbuf, dres, &gin, s);
        if (e != hipSuccess) return e;
    }
    if (g_used) *g_used = gin;
    return launch_mfma_dgrad_prepared(g, gin, scale, w, dx, accumulate, ws, ws_bytes, s, later);
}

// ---- fused backward -------------------------------------------------------------------------
// Packs the flipped, scaled weights into ws and, in the same launch, forms g = dy*[y>0] in the two
// layouts the gradients read: plain (into dres when the caller wants the residual gradient, else into
// the workspace behind the packed weights; skipped when there is no ReLU and no dres) and in fragment
// order (gf).  *g_plain receives the tensor the input-gradient engine has to contract.  Rows of any length: g is
// always formed, pitched, in the workspace; gf is optional; x (optional) is copied to xp in the same launch.
hipError_t launch_bwd_prepare(const Geom &g, const void *dy, const void *y, const float *scale, const void *w,
                              bool pack, bool relu, void *ws, void *gf, const DzfLayout &layout, void *dres, const void **g_plain,
                              hipStream_t s, const void *x, void *xp)
{
    if (!rows16(g)) {
        RowPrep a = {};
        a.w = pack ? w : nullptr;
        a.wp = ws;
        a.flip = true;
        a.rscale = scale;
        a.dy = dy;
        a.y = y;
        a.relu = relu;
        a.gplain = (unsigned char *)ws + packed_bytes(g.Cin, g.Cout, g.K);
        a.dres = dres;
        a.gf = gf;
        a.ncm = layout.ncm;
        a.nst = layout.nst;
        a.x = g.T % 8 == 0 ? nullptr : x;
        a.xp = xp;
        *g_plain = a.gplain;
        return launch_prepare_rows(g, a, s);
    }
    const int M = g.Cin, R = g.Cout;  // the engine's roles for the input gradient
    PackGeom q = pack_geom(w, M, R, g.K, true);
    if (!pack) q.blocks = 0, q.lds = 0;
    const size_t nfrag = (size_t)g.B * layout.ncm * ((layout.nst + 3) / 4);  // items of four fragments, one per wavefront
    void *gbuf = (unsigned char *)ws + packed_bytes(g.Cin, g.Cout, g.K);
    void *gout = dres ? dres : (relu ? gbuf : nullptr);
    *g_plain = gout ? gout : dy;
    static LdsOptIn opt_in;
    hipError_t e = ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(bwd_prepare_kernel), kMaxLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bwd_prepare_kernel, dim3(q.blocks + (unsigned)((nfrag + 3) / 4)), dim3(256), q.lds, s, q.blocks,
                       (const bf16_t *)w, (u32x4 *)ws, M, R, g.K, q.nch, M * g.K, q.zero_off, q.vec, scale, g.B, g.Cout, g.To,
                       layout.ncm, layout.nst, (const bf16_t *)dy, (const bf16_t *)y, relu ? 1 : 0, (u32x4 *)gout, (u32x4 *)gf);
    return hipGetLastError();
}

hipError_t launch_mfma_dgrad_prepared(const Geom &g, const void *g_plain, const float *scale, const void *w, void *dx, bool accumulate,
                                      void *ws, size_t ws_bytes, hipStream_t s, SplitSum *later)
{
    const Plan pl = make_plan(row_pitch(g.To), g.T, g.Cout, g.K, 1, g.dil);
    if (!pl.ok || !mfma_dgrad_supported(g)) return hipErrorInvalidValue;
    ConvGemmParams p = {};
    fill_dgrad(p, pl, g, g_plain, ws, dx, accumulate);
    const size_t least = mfma_dgrad_workspace_least(g);
    if (mfma_dgrad_unpacked(g, w, ws_bytes))
        return launch_unpacked_conv(dgrad_unpacked_plan(g, pl, ws_bytes), p, w, true, scale, (unsigned char *)ws + least, s, later);
    return launch_plan(pl, dgrad_split_plan(g, pl, ws_bytes), p, s, (unsigned char *)ws + least, ws_bytes - least, later);
}

}  // namespace nm
