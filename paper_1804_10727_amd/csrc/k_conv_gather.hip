// Output rows of a convolution of any kernel size, stride and padding on the matrix cores: every lane
// gathers the cells of its own window from memory.
//
// A layer keeps the rows of its input that some output row still needs, as events, in a ring; an output
// row is formed in registers once its last input row has arrived, activated and emitted into the ring of
// the next layer.  A launch holds a step for every layer that has rows to form, all on rows that
// were complete before it, and one that puts the caller's new rows into the first ring.
//
// Max-pools, in nets that have them, are steps of the same launch.  Measured per image of 112 x 112, 32 streams, float32,
// six layers (5x5 and 3x3 with stride 2, 3x3, 1x1, a pool): 532 to 576 us, 4.9 per row; a launch per layer, the layers that are not
// 3x3 with stride 1 on the vector units: 4360, 39 per row.
//
// The work is a matrix product: the columns of the instruction are output positions -- of one stream, or, where
// a stream has few, of 2, 4, 8 or 16 streams side by side, so that a layer that completes four rows of a
// 1-D signal per push still fills its tiles -- its rows 16 output channels, and the contraction runs over
// the window's cells of 16 bytes, (ky, kx, cell of channels).  What a launch costs is latency, not
// arithmetic: the windows of 64 audio streams are 64 tiles for each of the deep layers.  So a tile goes
// to four waves, a quarter of the contraction each, which ask for everything they need (at most nine
// K-steps at a time) before they use any of it; their sums are added in a fixed order.  Results do not depend
// on how rows or streams were grouped.  K-steps whose 16 positions hold no event are skipped.
//
//   k_conv_gather_rows    a workgroup per tile, all steps side by side (_staged: some steps' windows by way of LDS);
//   k_conv_gather_chain   a workgroup of four such teams per stream, the steps one after the other: rows that
//                         are to come out at once go through all layers in one launch.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "idf.h"
#include "idf_kernels.h"
#include "mfma_tile.h"

namespace idf {

namespace {

typedef const __attribute__((address_space(4))) GatherStep Step;
typedef const __attribute__((address_space(4))) GatherHead Head;

constexpr int kTeam = 4;                         // waves that share a tile
constexpr int kChunk = 9;                        // K-steps a wave has in flight
constexpr int kStages = 2;                       // and a wave of a tile of two by two (with 3, or 5 at once: one wave per SIMD less, which costs more)
constexpr int kPoolCells = 64 * kTeam;           // cells of a pool's rows per workgroup
constexpr int kStageCells = 1280, kStageLoads = 4;   // cells of windows in LDS; loads of a lane that bring them

// Cells in LDS from one stream's rows to the next's.  The positions of two streams (four each; or eight of one) are served together:
// they lie on banks of their own where all their distances are even and none the same (cells mod 16).
__host__ __device__ inline int stage_block(int rows, int pitch, int s_h_log)
{
    const int n = rows * pitch, want = s_h_log == 0 ? 8 : 2;
    return n + ((want - n) & 15);
}

// Taps of an axis that position v lands on inside an output of n positions (n == 0: unbounded).
__device__ __forceinline__ int taps_axis(int v, int k, int s_log, int p, int n)
{
    int hi = (v + p) >> s_log;
    int lo = (v + p - k + (1 << s_log)) >> s_log;
    lo = lo < 0 ? 0 : lo;
    if (n > 0 && hi >= n) hi = n - 1;
    return hi >= lo ? hi - lo + 1 : 0;
}

// The sum over the four lanes that are 16 apart, in each of them.
__device__ __forceinline__ uint32_t other_halves(uint32_t v)
{
    auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = r[0] + r[1];
    r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return r[0] + r[1];
}

// ---- the caller's rows: into the ring, channels padded to whole cells, and counted as the first layer's events ----
template <class T> __device__ __forceinline__ void take_rows(Head &h, Step &a, const StreamSel &sel, int si, int tid, int threads)
{
    using ev_t = typename T::ev_t;
    const int stream = sel_stream(sel, si), lane = tid & 63;
    // (a pixel segment brings x_n columns of its row, from x0 on)
    const int c_in = a.c_in, cells = a.cells, n_rows = a.n_rows, seg_rows = h.seg_rows, x0 = a.dst_slot0, x_n = a.dst_rows;
    const int row_elems = x_n * c_in, row_cells = x_n * cells, ring_cells = a.w_in * cells;
    unsigned char *ring = (unsigned char *)a.ring + (int64_t)stream * a.ring_stride * T::EB;
    uint32_t ev = 0, taps = 0;
    for (int i = tid; i < n_rows * row_cells; i += threads) {
        const int r = row_cells == 1 ? i : i / row_cells, xc = i - r * row_cells, x = cells == 1 ? xc : xc / cells, c = (xc - x * cells) * T::VL;
        const int seg = h.n_in == 1 ? 0 : r / seg_rows;
        // (the pointer of a lane's own buffer: from the arguments, by a vector load)
        const ev_t *src = (const ev_t *)((const __attribute__((address_space(4))) uint64_t *)h.in)[seg] +
                          (int64_t)(sel.pos0 + si) * h.in_stride + (r - seg * seg_rows) * row_elems + x * c_in + c;
        ev_t v[T::VL];
        uint32_t n = 0;
#pragma unroll
        for (int e = 0; e < T::VL; ++e) v[e] = c + e < c_in ? src[e] : (ev_t)0;
#pragma unroll
        for (int e = 0; e < T::VL; ++e) n += T::ev_nonzero(v[e]);
        i32x4 cell;
        __builtin_memcpy(&cell, v, 16);
        int slot = a.slot0 + r;
        slot = slot >= a.ring_rows ? slot - a.ring_rows : slot;
        *at4(reinterpret_cast<i32x4 *>(ring), (uint32_t)(slot * ring_cells + x0 * cells + xc) * 16) = cell;
        ev += n;
        taps += n * (uint32_t)(taps_axis(a.y0 + r, a.k_h, a.s_h_log, a.p_h, a.h_out) * (a.flat ? 1 : taps_axis(x0 + x, a.k_w, a.s_w_log, a.p_w, a.w_out)));
    }
    if (!h.stats) return;
    ev = wave_sum(ev); taps = wave_sum(taps);
    if (lane == 0 && ev) {
        unsigned long long *d = h.stats + ((int64_t)stream * h.n_layers + a.layer) * 2;
        atomicAdd(d, (unsigned long long)ev);
        atomicAdd(d + 1, (unsigned long long)taps * (unsigned long long)a.c_out);
    }
}

// ---- max-pool: rows of the layer's ring into the next one, a cell of 16 bytes per thread ---------------------
template <class T> __device__ __forceinline__ void pool_rows(Head &h, Step &a, const StreamSel &sel, int si, int first, int past, int threads)
{
    using ev_t = typename T::ev_t;
    const int stream = sel_stream(sel, si), lane = threadIdx.x & 63;
    const int cells = a.cells, k_w = a.k_w, w_in = a.w_in, w_out = a.w_out, row_cells = w_out * cells, items = a.n_rows * row_cells;
    const i32x4 *ring = reinterpret_cast<const i32x4 *>((const unsigned char *)a.ring + (int64_t)stream * a.ring_stride * T::EB);
    i32x4 *dst = reinterpret_cast<i32x4 *>((unsigned char *)a.dst + (int64_t)stream * a.dst_stride * T::EB);
    auto val = [](ev_t v) IDF_INLINE {
        if constexpr (T::EB == 2) return __uint_as_float((uint32_t)v << 16);
        else return v;
    };
    auto larger = [&](i32x4 u, i32x4 v) IDF_INLINE {
        ev_t p[T::VL], q[T::VL];
        __builtin_memcpy(p, &u, 16);
        __builtin_memcpy(q, &v, 16);
#pragma unroll
        for (int e = 0; e < T::VL; ++e) p[e] = val(p[e]) > val(q[e]) ? p[e] : q[e];
        __builtin_memcpy(&u, p, 16);
        return u;
    };
    uint32_t ev = 0, taps = 0;
    for (int i = first + (int)threadIdx.x; i < past && i < items; i += threads) {
        const int r = i / row_cells, xc = i - r * row_cells, x = xc / cells, c = xc - x * cells;
        int s0 = a.slot0 + 2 * r, s1 = s0 + 1;
        s0 = s0 >= a.ring_rows ? s0 - a.ring_rows : s0;
        s1 = s1 >= a.ring_rows ? s1 - a.ring_rows : s1;
        const int at0 = (s0 * w_in + x * k_w) * cells + c, at1 = (s1 * w_in + x * k_w) * cells + c;
        i32x4 m = larger(ring[at0], ring[at1]);
        if (k_w == 2) m = larger(larger(ring[at0 + cells], ring[at1 + cells]), m);
        int slot = a.dst_slot0 + r;
        slot = slot >= a.dst_rows ? slot - a.dst_rows : slot;
        dst[slot * row_cells + xc] = m;
        uint32_t n = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) n += (uint32_t)T::nonzero((uint32_t)m[q]);
        ev += n;
        taps += n * (uint32_t)(taps_axis(a.y0 + r, a.nk_h, a.ns_h_log, a.np_h, a.nh_out) * taps_axis(x, a.nk_w, a.ns_w_log, a.np_w, a.nw_out));
    }
    if (!h.stats) return;
    ev = wave_sum(ev); taps = wave_sum(taps);
    if (lane == 0 && ev) {
        unsigned long long *d = h.stats + ((int64_t)stream * h.n_layers + a.next_layer) * 2;
        atomicAdd(d, (unsigned long long)ev);
        atomicAdd(d + 1, (unsigned long long)taps * (unsigned long long)a.next_c_out);
    }
}

// ---- one tile: 16 positions x 16 channels, by a team of four waves ---------------------------------------
// What a launch of few tiles spends its time on is what stands around the contraction: a wave's arguments in one batch (and asked for
// in one statement: request_arguments), cells found with an addition and two minima where they lie in one stretch, counters
// added over lanes without LDS, in one instruction (us: 64 audio streams 5898 -> 5548 per 16,000 samples, one live stream 32.2 -> 29.2
// per segment, 37 streams with 16 pushes per launch 741 -> 713, 32 images through six layers 565 -> 532; one sensor, whose pushes wait
// for the host, the same).  Taken out again one by one: counters by exchanges through LDS 5643 -> 5832 and 29.5 -> 30.3; a statement per
// requested line 5683 and 29.6, no batch 5589 and 29.6, which is nothing: what is left is the way to the cells.
// TW 2: two such tiles of channels x two of positions.  Their sums are those of single tiles, formed in the same order; each weight
// and each cell that is fetched serves two tiles, and each wave brings one of the four to its end.
// share: LDS for the waves' sums (three, or four per tile); barrier: where the team's waves meet.
template <class T, bool COUNT, bool CHAIN, int TW, bool STAGE, class Barrier>
__device__ __forceinline__ void conv_tile(Head &h, Step &a, const StreamSel &sel, int si0, int pt, int ct, int spt_log, bool on, int kq,
                                          typename T::acc_t *share, i32x4 *cells_at, Barrier &&barrier)
{
    using acc_t = typename T::acc_t; using st_t = typename T::st_t;
    constexpr int VL = T::VL, EB = T::EB, NT = TW * TW;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    // everything the tile needs to know, asked for in one batch (left to first use: one wait after the other)
    const int n_rows = a.n_rows, y0 = a.y0, n_ks = a.n_ks, cells = a.cells, slot0 = a.slot0, ring_rows = a.ring_rows, k_h = a.k_h, s_h_log = a.s_h_log;
    const int64_t ring_stride = a.ring_stride, dst_stride = a.dst_stride;
    const void *ring_p = a.ring, *w_frag = a.w_frag;
    void *dst = a.dst;
    const st_t *bias = (const st_t *)a.bias;
    const int h_in = a.h_in, p_h = a.p_h, n_ct = a.n_ct, flat = a.flat, w_out = a.w_out;
    const int act = a.act, shr = a.shr, clamp_hi = a.clamp_hi, c_out = a.c_out, dst_cells = a.dst_cells, dst_slot0 = a.dst_slot0, dst_rows = a.dst_rows;
    const int next_layer = a.next_layer, nk_h = a.nk_h, ns_h_log = a.ns_h_log, np_h = a.np_h, nh_out = a.nh_out, next_c_out = a.next_c_out, to_output = a.to_output;
    unsigned long long *stats = h.stats;
    const int n_layers = h.n_layers;
    asm volatile("" ::"s"(n_rows), "s"(y0), "s"(n_ks), "s"(cells), "s"(slot0), "s"(ring_rows), "s"(k_h), "s"(s_h_log), "s"(ring_stride), "s"(ring_p), "s"(w_frag),
                 "s"(h_in), "s"(p_h), "s"(n_ct), "s"(flat), "s"(w_out));
    // (for what comes after the contraction; where steps follow each other in a loop that many registers are not free until then)
    auto later = [&]() IDF_INLINE {
        asm volatile("" ::"s"(act), "s"(shr), "s"(clamp_hi), "s"(c_out), "s"(dst_cells), "s"(dst_slot0), "s"(dst_rows), "s"(next_layer), "s"(nk_h), "s"(ns_h_log),
                     "s"(np_h), "s"(nh_out), "s"(next_c_out), "s"(to_output), "s"(stats), "s"(n_layers), "s"(dst_stride), "s"(dst), "s"(bias));
    };
    if (!CHAIN) later();
    const int per_log = 4 - spt_log;               // positions per stream in the tile
    const int si = si0 + (m >> per_log), pl = m & ((1 << per_log) - 1);
    const bool stream_ok = on && si < sel.n;
    const int stream = sel_stream(sel, stream_ok ? si : 0);
    const unsigned char *ring = (const unsigned char *)ring_p + (int64_t)stream * ring_stride * EB;
    const uint32_t lane16 = (uint32_t)lane * 16, w_step = (uint32_t)n_ct * 1024;
    // this wave's K-steps
    const int each = (n_ks + kTeam - 1) / kTeam, ks0 = kq * each, ks1 = ks0 + each < n_ks ? ks0 + each : n_ks;
    const unsigned char *wf0[TW];
#pragma unroll
    for (int tc = 0; tc < TW; ++tc) wf0[tc] = (const unsigned char *)w_frag + (TW == 1 || ct + tc < n_ct ? ct + tc : ct) * 1024 + ks0 * w_step;
    // a lane's position in a tile: row and column of the output
    auto place = [&](int tp, int &o, int &x) IDF_INLINE {
        const int p = ((pt * TW + tp) << per_log) + pl;
        o = p; x = 0;
        if (!flat) { o = w_out == 1 ? p : (int)__umulhi((unsigned)p, a.wout_rcp); x = p - o * w_out; }
        const bool valid = stream_ok && o < n_rows;
        o = valid ? o : 0;
        return valid;
    };
    int o = 0, x = 0;
    bool valid = false;
    // A K-step's instructions have sums of their own: none waits for the one before, and the chains that round are a quarter as long.
    acc_t sums[T::kInst][NT] = {}, acc = {0, 0, 0, 0};
    if (on) {
        bool there_is[TW];
        int y_in[TW];                              // the window's first row
        unsigned slot_o[TW];
        int x_of[TW];
#pragma unroll
        for (int tp = 0; tp < TW; ++tp) {
            there_is[tp] = place(tp, o, x);
            x_of[tp] = x;
            y_in[tp] = ((y0 + o) << s_h_log) - p_h;
            slot_o[tp] = (unsigned)(slot0 + (o << s_h_log));
            slot_o[tp] = min(slot_o[tp], slot_o[tp] - (unsigned)ring_rows);
        }
        valid = there_is[0];
        if constexpr (TW > 1) {
            // (tiles of one stream: a lane's place outside the map or the window is a place outside the ring, where nothing is read and
            // zeros come back.  The next K-steps are on their way while one is multiplied; what bounds it is the L2, which every
            // workgroup asks for all weights of its channels: without any contraction a launch of 37 audio streams with 16 pushes each
            // takes 5.5 us under the profiler, without its matrix instructions 16.5, in all 17.6; single tiles 22.6)
            const int k_w = flat ? 1 : a.k_w, row_cells = flat ? cells : a.w_in * cells, win_cells = k_w * cells;
            const unsigned win_rcp = a.win_rcp, one = win_cells == 1;
            const uint32_t ring_bytes = (uint32_t)(ring_rows * row_cells) * 16;
            unsigned char *first = (unsigned char *)const_cast<void *>(ring_p) + (int64_t)sel_stream(sel, si0) * ring_stride * EB;
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(first, 0, (int)ring_bytes, 0x00027000);
            uint32_t begin[TW], n_q[TW];           // flat: cells of the window inside the signal, from q_lo on
            int q_lo[TW], xc0[TW];
#pragma unroll
            for (int tp = 0; tp < TW; ++tp) {
                q_lo[tp] = max(0, -y_in[tp]) * cells;
                n_q[tp] = there_is[tp] ? (uint32_t)(min(k_h, h_in - y_in[tp]) * cells - q_lo[tp]) : 0u;
                begin[tp] = slot_o[tp] * (uint32_t)cells * 16;
                xc0[tp] = flat ? 0 : ((x_of[tp] << a.s_w_log) - a.p_w) * cells;
            }
            const int q_end = k_h * win_cells;
            i32x4 xv[kStages][TW], wv[kStages][TW];
            auto fetch = [&](i32x4 (&x_s)[TW], i32x4 (&w_s)[TW], int ks) IDF_INLINE {
                ks = ks < ks1 ? ks : ks1 - 1;      // (past the end the last one again)
#pragma unroll
                for (int tc = 0; tc < TW; ++tc) w_s[tc] = *at4(reinterpret_cast<const i32x4 *>(wf0[tc] + (ks - ks0) * w_step), lane16);
                const int q = 4 * ks + g;
                const unsigned ky = flat ? 0u : __umulhi((unsigned)q, win_rcp) + __umul24((unsigned)q, one);
#pragma unroll
                for (int tp = 0; tp < TW; ++tp) {
                    uint32_t off;
                    bool ok;
                    if (flat) {
                        off = begin[tp] + (uint32_t)q * 16;
                        off = min(off, off - ring_bytes);
                        ok = (uint32_t)(q - q_lo[tp]) < n_q[tp];
                    } else {
                        const int xc = xc0[tp] + q - (int)__umul24(ky, (unsigned)win_cells);
                        unsigned slot = slot_o[tp] + ky;
                        slot = min(slot, slot - (unsigned)ring_rows);
                        slot = min(slot, slot - (unsigned)ring_rows);
                        off = (__umul24(slot, (unsigned)row_cells) + (unsigned)xc) * 16;
                        ok = there_is[tp] && (unsigned)y_in[tp] + ky < (unsigned)h_in && (unsigned)xc < (unsigned)row_cells && q < q_end;
                    }
                    x_s[tp] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, ok ? (int)off : INT32_MIN, 0, 0));
                }
            };
            auto contract = [&](const i32x4 (&x_s)[TW], const i32x4 (&w_s)[TW]) IDF_INLINE {
#pragma unroll
                for (int tp = 0; tp < TW; ++tp) {
                    if (__ballot(T::or_of(x_s[tp]) != 0) == 0ull) continue;
#pragma unroll
                    for (int e = 0; e < T::kInst; ++e)
#pragma unroll
                        for (int tc = 0; tc < TW; ++tc) sums[e][tp * TW + tc] = T::mfma(w_s[tc], x_s[tp], sums[e][tp * TW + tc], e);
                }
            };
            if (ks0 < ks1) {                       // (short windows leave a wave without a K-step)
#pragma unroll
                for (int i = 0; i < kStages; ++i) fetch(xv[i], wv[i], ks0 + i);
                int ks = ks0;
#pragma unroll 1
                for (; ks + kStages < ks1; ks += kStages) {
#pragma unroll
                    for (int i = 0; i < kStages; ++i) {
                        contract(xv[i], wv[i]);
                        fetch(xv[i], wv[i], ks + kStages + i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // (the last ones stand behind the loop: nothing is asked for that no K-step is left for.  Three requests of twelve in a wave
                // with nine K-steps were; a launch of 37 audio streams with 16 pushes each 13.4 -> 12.5 us, of 64 18.5 -> 17.1)
#pragma unroll
                for (int i = 0; i < kStages; ++i)
                    if (ks + i < ks1) contract(xv[i], wv[i]);
            }
        } else {
            unsigned long long issued = 0;
            auto contract = [&](const i32x4 (&xv)[kChunk], const i32x4 (&wv)[kChunk], int kb) IDF_INLINE {
#pragma unroll
                for (int i = 0; i < kChunk; ++i) {
                    if (kb + i >= ks1) continue;
                    if (__ballot(T::or_of(xv[i]) != 0) == 0ull) continue;
#pragma unroll
                    for (int e = 0; e < T::kInst; ++e) sums[e][0] = T::mfma(wv[i], xv[i], sums[e][0], e);
                    if (COUNT) {
                        const int n_cells = k_h * (flat ? 1 : a.k_w) * cells;
                        for (int u = 0; u < 4; ++u) {
                            const int q = 4 * (kb + i) + u, c = q % cells;
                            if (q < n_cells) issued += (a.c_in - c * VL < VL ? a.c_in - c * VL : VL);
                        }
                    }
                }
            };
            if constexpr (STAGE) {
                // The rows that the tile's windows lie in go to LDS once, those of each stream by 4 / streams waves: windows that follow one
                // another share all but their first rows, and loads of single cells are what bounds a launch of many tiles.
                const int streams_log = 4 - per_log, cells_log = 31 - __builtin_clz(cells), P = 1 << per_log;
                const int rows = ((P - 1) << s_h_log) + k_h, pitch = cells + 2, block = stage_block(rows, pitch, s_h_log);
                const int own = kq >> (2 - streams_log), n = rows << cells_log;
                const int y_first = ((y0 + (pt << per_log)) << s_h_log) - p_h;
                const bool there = si0 + own < sel.n;
                const unsigned char *from = (const unsigned char *)ring_p + (int64_t)sel_stream(sel, there ? si0 + own : 0) * ring_stride * EB;
                i32x4 wv[kChunk], cv[kStageLoads];
                const unsigned char *wf = wf0[0];
#pragma unroll
                for (int i = 0; i < kChunk; ++i)
                    if (ks0 + i < ks1) wv[i] = *at4(reinterpret_cast<const i32x4 *>(wf), (uint32_t)i * w_step + lane16);
                const int i0 = (kq & ((4 >> streams_log) - 1)) * 64 + lane, step = 256 >> streams_log;
#pragma unroll
                for (int j = 0; j < kStageLoads; ++j) {
                    const int i = i0 + j * step, r = i >> cells_log;
                    unsigned slot = (unsigned)(slot0 + (((pt << per_log)) << s_h_log) + r);
                    slot = min(slot, slot - (unsigned)ring_rows);
                    slot = min(slot, slot - (unsigned)ring_rows);
                    const bool ok = i < n && there && (unsigned)(y_first + r) < (unsigned)h_in;
                    cv[j] = i32x4{0, 0, 0, 0};
                    if (ok) cv[j] = *at4(reinterpret_cast<const i32x4 *>(from), (slot << cells_log | (unsigned)(i & (cells - 1))) * 16);
                }
#pragma unroll
                for (int j = 0; j < kStageLoads; ++j) {
                    const int i = i0 + j * step;
                    if (i < n) cells_at[own * block + (i >> cells_log) * pitch + (i & (cells - 1))] = cv[j];
                }
                lds_barrier();
                const i32x4 *mine = cells_at + (m >> per_log) * block + (pl << s_h_log) * pitch + g;
#pragma unroll 1
                for (int kb = ks0; kb < ks1; kb += kChunk) {
                    i32x4 xv[kChunk];
                    if (kb > ks0) {
#pragma unroll
                        for (int i = 0; i < kChunk; ++i)
                            if (kb + i < ks1) wv[i] = *at4(reinterpret_cast<const i32x4 *>(wf0[0] + (kb - ks0) * w_step), (uint32_t)i * w_step + lane16);
                    }
#pragma unroll
                    for (int i = 0; i < kChunk; ++i) {
                        if (kb + i >= ks1) continue;
                        const int q = 4 * (kb + i);
                        xv[i] = mine[(q >> cells_log) * pitch + (q & (cells - 1))];
                        if (!valid) xv[i] = i32x4{0, 0, 0, 0};
                    }
                    contract(xv, wv, kb);
                }
            } else if (flat) {
                const int q_last = k_h * cells - 1;
                // (a window that reaches over an end of the signal: its cells there are zero; so are those past the window's end, where
                // the weights are zero too, but zero times infinity is not)
                const bool edge = __ballot(valid && (y_in[0] < 0 || y_in[0] + k_h > h_in)) != 0ull || 4 * n_ks > q_last + 1;
                // a position's rows follow each other in the ring and have nothing between them: the window is one stretch, but for the
                // ring's end (cells past the window's end: see above, the last one again)
                const uint32_t ring_bytes = (uint32_t)(ring_rows * cells) * 16, begin = slot_o[0] * (uint32_t)cells * 16, last = (uint32_t)q_last * 16;
                const unsigned cells_rcp = a.cells_rcp;
#pragma unroll 1
                for (int kb = ks0; kb < ks1; kb += kChunk) {
                    i32x4 xv[kChunk], wv[kChunk];
                    const unsigned char *wf = wf0[0] + (kb - ks0) * w_step;
                    const uint32_t at = (uint32_t)(4 * kb + g) * 16;
#pragma unroll
                    for (int i = 0; i < kChunk; ++i) {
                        if (kb + i >= ks1) continue;
                        wv[i] = *at4(reinterpret_cast<const i32x4 *>(wf), (uint32_t)i * w_step + lane16);
                        uint32_t off = begin + min(at + (uint32_t)i * 64, last);
                        off = min(off, off - ring_bytes);
                        xv[i] = *at4(reinterpret_cast<const i32x4 *>(ring), off);
                    }
                    if (edge) {
#pragma unroll
                        for (int i = 0; i < kChunk; ++i) {
                            if (kb + i >= ks1) continue;
                            const int q = 4 * (kb + i) + g, y = y_in[0] + (int)(__umul24((unsigned)q, cells_rcp) >> 16);
                            if (y < 0 || y >= h_in || q > q_last) xv[i] = i32x4{0, 0, 0, 0};
                        }
                    }
                    if (!valid) {
#pragma unroll
                        for (int i = 0; i < kChunk; ++i) if (kb + i < ks1) xv[i] = i32x4{0, 0, 0, 0};
                    }
                    contract(xv, wv, kb);
                }
            } else {
                // likewise a row of the window, k_w positions; what lies outside the row is outside of both ends of its cells
                const int k_w = a.k_w, w_in = a.w_in, row_cells = w_in * cells, win_cells = k_w * cells, x_in = ((x << a.s_w_log) - a.p_w) * cells, q_last = k_h * win_cells - 1;
                const unsigned win_rcp = a.win_rcp, one = win_cells == 1;
#pragma unroll 1
                for (int kb = ks0; kb < ks1; kb += kChunk) {
                    i32x4 xv[kChunk], wv[kChunk];
                    const unsigned char *wf = wf0[0] + (kb - ks0) * w_step;
                    uint32_t there = 0;
#pragma unroll
                    for (int i = 0; i < kChunk; ++i) {
                        if (kb + i >= ks1) continue;
                        wv[i] = *at4(reinterpret_cast<const i32x4 *>(wf), (uint32_t)i * w_step + lane16);
                        const unsigned q = (unsigned)(4 * (kb + i) + g), ky = __umulhi(q, win_rcp) + __umul24(q, one);
                        const int xc = x_in + (int)(q - __umul24(ky, (unsigned)win_cells));
                        const bool ok = valid && (unsigned)y_in[0] + ky < (unsigned)h_in && (unsigned)xc < (unsigned)row_cells && (int)q <= q_last;
                        there |= ok ? 1u << i : 0u;
                        unsigned slot = slot_o[0] + ky;
                        slot = min(slot, slot - (unsigned)ring_rows);
                        slot = min(slot, slot - (unsigned)ring_rows);
                        xv[i] = *at4(reinterpret_cast<const i32x4 *>(ring), ok ? (__umul24(slot, (unsigned)row_cells) + (unsigned)xc) * 16 : 0u);
                    }
#pragma unroll
                    for (int i = 0; i < kChunk; ++i)
                        if (kb + i < ks1 && !((there >> i) & 1u)) xv[i] = i32x4{0, 0, 0, 0};
                    contract(xv, wv, kb);
                }
            }
            if (COUNT && h.issued && g == 0 && pl == 0 && si < sel.n && issued) {
                const int co_n = a.c_out - ct * 16 < 16 ? a.c_out - ct * 16 : 16;
                atomicAdd(h.issued + (int64_t)sel_stream(sel, si) * h.n_layers + a.layer, (issued * (unsigned long long)co_n) << per_log);
            }
        }
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if constexpr (T::kInst == 4) acc = (sums[0][i] + sums[1][i]) + (sums[2][i] + sums[3][i]);
            else acc = sums[0][i];
            if (TW > 1) share[(i * kTeam + kq) * 64 + lane] = acc;
            else if (kq > 0) share[(kq - 1) * 64 + lane] = acc;
        }
    }
    if (CHAIN) later();
    barrier();
    if (!on || (TW == 1 && kq > 0)) return;
    if (TW > 1) {                                  // this wave's tile
        if (ct + (kq & 1) >= n_ct) return;
        ct += kq & 1;
        valid = place(kq >> 1, o, x);
    }

    const int co0 = ct * 16 + g * 4;
    st_t hv[4];
    {
        acc_t part[kTeam - 1];
        if (TW > 1) acc = share[kq * kTeam * 64 + lane];
#pragma unroll
        for (int w = 0; w < kTeam - 1; ++w) part[w] = share[(TW > 1 ? kq * kTeam + 1 + w : w) * 64 + lane];
        st_t c[4] = {0, 0, 0, 0};
        if (bias) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = bias[co0 + i < c_out ? co0 + i : c_out - 1];
        }
        acc = (acc + part[0]) + (part[1] + part[2]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c[i] += acc[i];
            hv[i] = co0 + i < c_out ? T::activate(c[i], act, shr, clamp_hi) : (st_t)0;
        }
    }
    // steps one after the other: this one's rows are there before the wave goes on.  (Its counters need not be.)
    auto settle = [&]() IDF_INLINE {
        if constexpr (CHAIN) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    int slot = dst_slot0 + o;
    slot = slot >= dst_rows ? slot - dst_rows : slot;
    const int at = flat ? slot : slot * w_out + x;
    if (to_output) {                               // 4-byte values, not rounded to the event type
        st_t *d = (st_t *)dst + (int64_t)stream * dst_stride + (int64_t)at * c_out + co0;
        if (valid) {
            if (c_out % 4 == 0) {
                if (co0 < c_out) *reinterpret_cast<acc_t *>(d) = acc_t{hv[0], hv[1], hv[2], hv[3]};
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (co0 + i < c_out) d[i] = hv[i];
            }
        }
        settle();
        return;
    }
    uint32_t e[EB], nz = 0;
    T::pack4(hv, e);
    if (valid && co0 < dst_cells * VL) {
        unsigned char *d = (unsigned char *)dst + ((int64_t)stream * dst_stride + (int64_t)at * dst_cells * VL + co0) * EB;
        if constexpr (EB == 1) *reinterpret_cast<uint32_t *>(d) = e[0];
        else if constexpr (EB == 2) *reinterpret_cast<i32x2 *>(d) = i32x2{(int)e[0], (int)e[1]};
        else *reinterpret_cast<i32x4 *>(d) = i32x4{(int)e[0], (int)e[1], (int)e[2], (int)e[3]};
#pragma unroll
        for (int i = 0; i < EB; ++i) nz += (uint32_t)T::nonzero(e[i]);
    }
    if (!stats || next_layer < 0) {
        settle();
        return;
    }
    // events of the next layer (at most 256: the low 12 bits) and the taps they reach, per stream: over the four groups of channels,
    // then over the stream's positions.  Two lanes add them, with one instruction.
    uint32_t sum = nz | nz * (uint32_t)(taps_axis(y0 + o, nk_h, ns_h_log, np_h, nh_out) * (flat ? 1 : taps_axis(x, a.nk_w, a.ns_w_log, a.np_w, a.nw_out))) << 12;
    sum = other_halves(sum);
    if (per_log > 0) sum += (uint32_t)__builtin_amdgcn_mov_dpp((int)sum, 0xB1, 0xf, 0xf, true);        // lane ^ 1
    if (per_log > 1) sum += (uint32_t)__builtin_amdgcn_mov_dpp((int)sum, 0x4E, 0xf, 0xf, true);        // lane ^ 2
    if (per_log > 2) sum += (uint32_t)__builtin_amdgcn_mov_dpp((int)sum, 0x141, 0xf, 0xf, true);       // the other four of eight (mirrored)
    if (per_log > 3) sum += (uint32_t)__builtin_amdgcn_mov_dpp((int)sum, 0x140, 0xf, 0xf, true);       // the other eight of sixteen
    settle();
    if (g < 2 && pl == 0 && sum)
        atomicAdd(stats + ((int64_t)stream * n_layers + next_layer) * 2 + g, g == 0 ? (unsigned long long)(sum & 0xfffu) : (unsigned long long)(sum >> 12) * (unsigned)next_c_out);
}

// Workgroups that request the launch's arguments; those behind the first round find them in the scalar cache.  us, nobody asking /
// the first 256 / the first 512 / all: 64 audio streams 6090 / 5980 / 5785 / 5732; 37 streams with 16 pushes per launch 742 / 738 /
// 738 / 762; 32 images through six layers 606 / 583 / 551 / 615; one live stream 36.3, asking 32.2.
constexpr int kFirst = 512;
template <class T, int NS, bool COUNT, bool WIDE, bool STAGE> __device__ __forceinline__ void gather_rows(const StreamSel &sel)
{
    typedef const __attribute__((address_space(4))) GatherBatch<NS> Batch;
    Batch &b = *(Batch *)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ typename T::acc_t share[(WIDE ? 4 * kTeam : kTeam - 1) * 64];
    __shared__ i32x4 cells_at[STAGE ? kStageCells : 1];
    // The steps' tiles follow each other without gaps: workgroups go to the compute units in turn, and with an empty one here
    // and there some units got the tiles of three layers and others none (12.7 us per launch of 64 audio streams instead of 7).
    int k = 0, tile = blockIdx.x;
    if (blockIdx.x < kFirst) request_arguments<sizeof(Batch), kTeam>(&b, &b + 1);
    const int n_sb = b.head.n_sb, n_sb8 = b.head.n_sb8, sb_log = b.head.sb_log, n_sel = sel.n;
    const unsigned sb_rcp = b.head.sb_rcp;
    {
        int end[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) end[i] = b.head.end[i];
        const int base = sel.base, pos0 = sel.pos0;
        asm volatile("" ::"s"(end[0]), "s"(end[1]), "s"(end[2]), "s"(end[3]), "s"(end[4]), "s"(end[5]), "s"(end[6]), "s"(end[7]), "s"(n_sb), "s"(n_sb8), "s"(sb_log),
                     "s"(n_sel), "s"(sb_rcp), "s"(base), "s"(pos0));
        int first = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) if ((int)blockIdx.x >= end[i]) { k = i + 1; first = end[i]; }
        tile -= first;
    }
    Step &a = b.st[k];
    const int take = a.take, spt_log = a.spt_log;
    int sg, rest;                                  // group of streams; tile of positions and channels
    if (n_sb > 0) {
        // workgroups go to the XCDs in turn: a block of streams meets one and the same in every layer, whose L2 then has the
        // rows that the layer before has just written
        const int inner = (int)__umulhi((unsigned)tile, sb_rcp), sb = tile - inner * n_sb8, subs = sb_log - spt_log;
        if (sb >= n_sb) return;
        sg = (sb << subs) + (inner & ((1 << subs) - 1));
        rest = inner >> subs;
        if ((sg << spt_log) >= n_sel) return;
    } else {
        const int per = a.n_cg * a.n_pt;
        sg = take == 1 ? tile : (int)((unsigned)tile / (unsigned)per);
        rest = take == 1 ? 0 : tile - sg * per;
    }
    if (take == 1) { take_rows<T>(b.head, a, sel, sg, threadIdx.x, 64 * kTeam); return; }
    if (take == 2) { pool_rows<T>(b.head, a, sel, sg, rest * kPoolCells, (rest + 1) * kPoolCells, 64 * kTeam); return; }
    const int n_cg = a.n_cg, pt = a.ct_rcp ? (int)__umulhi((unsigned)rest, a.ct_rcp) : rest, cg = rest - pt * n_cg;
    const int wave = uni(threadIdx.x >> 6);
    if (WIDE && a.wide) conv_tile<T, COUNT, false, 2, false>(b.head, a, sel, sg, pt, 2 * cg, 0, true, wave, share, nullptr, [] { lds_barrier(); });
    else if (STAGE && a.wide) conv_tile<T, COUNT, false, 1, STAGE>(b.head, a, sel, sg << spt_log, pt, cg, spt_log, true, wave, share, cells_at, [] { lds_barrier(); });
    else conv_tile<T, COUNT, false, 1, false>(b.head, a, sel, sg << spt_log, pt, cg, spt_log, true, wave, share, nullptr, [] { lds_barrier(); });
}

template <class T, int NS, bool COUNT, bool WIDE>
__global__ void __launch_bounds__(64 * kTeam, 4) k_conv_gather_rows(const GatherBatch<NS> args, const StreamSel sel) { gather_rows<T, NS, COUNT, WIDE, false>(sel); }
template <class T, int NS>
__global__ void __launch_bounds__(64 * kTeam, 4) k_conv_gather_rows_staged(const GatherBatch<NS> args, const StreamSel sel) { gather_rows<T, NS, false, false, true>(sel); }

template <class T, int NS, bool COUNT>
__global__ void __launch_bounds__(256 * kTeam) k_conv_gather_chain(const GatherBatch<NS> args, const StreamSel sel)
{
    typedef const __attribute__((address_space(4))) GatherBatch<NS> Batch;
    Batch &b = *(Batch *)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ typename T::acc_t share[4][(kTeam - 1) * 64];
    request_arguments<sizeof(Batch), 4 * kTeam>(&b, &b + 1);
    const int team = uni(threadIdx.x >> 8), kq = uni((threadIdx.x >> 6) & 3), si = blockIdx.x;
    for (int k = 0; k < b.head.n; ++k) {
        Step &a = b.st[k];
        if (a.take == 1) {
            take_rows<T>(b.head, a, sel, si, threadIdx.x, 256 * kTeam);
            __syncthreads();                       // what this step stored is there for the next
        } else if (a.take == 2) {
            pool_rows<T>(b.head, a, sel, si, 0, INT32_MAX, 256 * kTeam);
            __syncthreads();
        } else {
            const int tasks = a.n_ct * ((a.n_rows * a.w_out + 15) >> 4);
            for (int t0 = 0; t0 < tasks; t0 += 4) {
                Step *step = &a;
                asm volatile("" : "+s"(step));     // (a tile's arguments are read anew: kept over the loop they do not fit the registers)
                const int t = t0 + team, pt = a.ct_rcp ? (int)__umulhi((unsigned)t, a.ct_rcp) : t, ct = t - pt * a.n_ct;
                conv_tile<T, COUNT, true, 1, false>(b.head, *step, sel, si, pt, ct, 0, t < tasks, kq, share[team], nullptr, [] { lds_barrier(); });
                lds_barrier();                     // the sums have been read, and every wave's rows are there for the next step
            }
        }
    }
}

// A workgroup per layer, stream by stream: a stream's new place may lie on what streams on one side of it held, so they go from that
// side, and a stream's rows are all read before one is written.  Once per change of the rows in use, not per push: a memory
// round trip per stream, 4 us for one, 25 us for 64 audio streams, 180 us for 512.
constexpr int kMoveThreads = 256;
__global__ void __launch_bounds__(kMoveThreads) k_ring_move(const RingMove a)
{
    const RingMove::Unit &u = a.unit[blockIdx.x];
    const int t = threadIdx.x, r = t / u.row_cells, c = t - r * u.row_cells;
    const bool mine = r < u.keep;
    const int64_t from = (int64_t)u.from_rows * u.row_cells, to = (int64_t)u.to_rows * u.row_cells;
    const int64_t src = (int64_t)((u.from_slot + r) % u.from_rows) * u.row_cells + c, dst = (int64_t)((u.to_slot + r) % u.to_rows) * u.row_cells + c;
    i32x4 *ring = (i32x4 *)u.ring, v = {0, 0, 0, 0};
    for (int i = 0; i < a.n; ++i) {
        const int64_t stream = a.first + (to > from ? a.n - 1 - i : i);
        if (mine) v = ring[stream * from + src];
        __syncthreads();
        if (mine) ring[stream * to + dst] = v;
        __syncthreads();
    }
}

// Positions of a step's tiles that belong to one stream.
int streams_per_tile_log(int positions, bool first)
{
    // (a first layer has few channels and its rows are many: its tiles stay with one stream)
    int l = 0;
    while (!first && l < 4 && (positions << (l + 1)) <= 16) ++l;
    return l;
}

// Tiles of a launch from which on they go two by two: a wave then fetches four operands for four products instead of eight, and
// all four waves bring a tile to its end, but a quarter of the workgroups has to fill the chip.  GPU time per pass, single tiles against
// two by two: audio net, 16 pushes per launch, 12 streams (1,536 tiles) 183 us against 184, 16 streams 213 : 191, 37 streams 374 : 299,
// 64 streams 546 : 406, but 8 streams 151 : 170; six-layer net, 4 rows per push, 64 images of 79 x 79 (some 1,500 tiles) float32
// 188 : 182, bfloat16 162 : 141, 15 images of 160 x 160 (700) 296 : 334 and 255 : 256.
// And where a sixteenth of them and more can: those of steps of 16 channels or few positions stay single, in a kernel that holds more LDS
// and a longer block of arguments.  Likewise, by the share that can: none, three 8-channel layers, 64 streams with 16 pushes per launch
// 315 : 325, four layers over images 79 wide, 4 rows per push, 128 images 292 : 298, bfloat16 260 : 264; 8 %, 64 and 128 images 240 : 237,
// 399 : 396 and 209 : 212, 335 : 327; 13 %, 184 : 185, 273 : 268 and 171 : 173, 243 : 238; a quarter, 50 images (400 of 1,650 tiles)
// 190 : 190 and 171 : 155.
constexpr int kWideTiles = 1536, kWideShare = 16;
bool wide_step(const GatherStep &a) { return a.take == 0 && a.n_ct >= 2 && a.n_pt >= 2 && a.spt_log == 0; }

// A step whose windows go through LDS: many K-steps, whole K-steps to a row, one to four streams per tile; and launches that have them
// do so from as many tiles on as there are compute units: with fewer it makes no difference.  us per pass, cell by cell : through LDS, audio
// net, 16 samples per push, 64 streams of 16,000 samples 5637 : 5323, of 8,000, 48 streams 2994 : 2818, 32 2584 : 2528, 16 (144 tiles)
// 2739 : 2733; 16 pushes per launch, 12 streams 302 : 298.  (Without any loads of cells the first would take 4888, without weights' 5455.)
bool stage_step(const GatherStep &a)
{
    if (a.take != 0 || !a.flat || a.spt_log > 2 || a.n_ks < 9 || a.cells < 4 || (a.cells & (a.cells - 1))) return false;
    const int P = 16 >> a.spt_log, rows = ((P - 1) << a.s_h_log) + a.k_h;
    return rows * a.cells <= kStageLoads * (256 >> a.spt_log) && stage_block(rows, a.cells + 2, a.s_h_log) << a.spt_log <= kStageCells && (P << a.s_h_log) + a.k_h <= a.ring_rows;
}
constexpr int kStageTiles = 256;

template <class T, int NS, bool WIDE, bool STAGE> hipError_t launch_ns(const GatherHead &h, const GatherStep *st, const StreamSel &sel, bool chain, const LaunchCtx &lc)
{
    GatherBatch<NS> b;
    b.head = h;
    // streams in blocks that no tile crosses, if there is one for every XCD
    b.head.sb_log = 2;
    for (int k = 0; k < h.n; ++k) b.head.sb_log = std::max(b.head.sb_log, st[k].spt_log);
    b.head.n_sb = (sel.n + (1 << b.head.sb_log) - 1) >> b.head.sb_log;
    b.head.n_sb8 = (b.head.n_sb + 7) / 8 * 8;
    if (b.head.n_sb * 5 < b.head.n_sb8 * 4) b.head.n_sb = 0;               // (blocks for at least four XCDs in five, in every round)
    b.head.sb_rcp = b.head.n_sb ? (unsigned)((0x100000000ull + b.head.n_sb8 - 1) / b.head.n_sb8) : 0u;
    int64_t tiles = 0;
    for (int k = 0; k < 8; ++k) b.head.end[k] = INT32_MAX;
    for (int k = 0; k < h.n; ++k) {
        b.st[k] = st[k];
        GatherStep &a = b.st[k];
        if (STAGE) a.wide = stage_step(a);
        if (WIDE && (a.wide = wide_step(a))) {
            a.n_cg = (a.n_ct + 1) / 2; a.n_pt = (a.n_pt + 1) / 2;
            a.ct_rcp = a.n_cg > 1 ? (unsigned)((0x100000000ull + a.n_cg - 1) / a.n_cg) : 0u;
        }
        const int groups = b.head.n_sb > 0 ? b.head.n_sb8 << (b.head.sb_log - a.spt_log) : (sel.n + (1 << a.spt_log) - 1) >> a.spt_log;
        a.tiles = groups * (a.take == 1 ? 1 : a.n_cg * a.n_pt);
        tiles += b.st[k].tiles;
        if (k < 8 && k + 1 < h.n) b.head.end[k] = (int)tiles;
    }
    if (chain) {
        const dim3 grid(sel.n), block(256 * kTeam);
        return h.issued ? launch(k_conv_gather_chain<T, NS, true>, grid, block, 0, lc, b, sel) : launch(k_conv_gather_chain<T, NS, false>, grid, block, 0, lc, b, sel);
    }
    if (tiles < 1 || tiles > INT32_MAX / (64 * kTeam)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(64 * kTeam);
    if constexpr (STAGE) return launch(k_conv_gather_rows_staged<T, NS>, grid, block, 0, lc, b, sel);
    else if constexpr (WIDE) return launch(k_conv_gather_rows<T, NS, false, true>, grid, block, 0, lc, b, sel);
    else return h.issued ? launch(k_conv_gather_rows<T, NS, true, false>, grid, block, 0, lc, b, sel) : launch(k_conv_gather_rows<T, NS, false, false>, grid, block, 0, lc, b, sel);
}

template <class T> hipError_t launch_t(const GatherHead &h, const GatherStep *st, const StreamSel &sel, bool chain, const LaunchCtx &lc)
{
    // tiles of two by two where there are so many that the chip is full with a quarter of them
    int64_t tiles = 0, paired = 0;
    for (int k = 0; k < h.n; ++k) {
        if (st[k].take != 0) continue;
        const int64_t n = (int64_t)((sel.n + (1 << st[k].spt_log) - 1) >> st[k].spt_log) * st[k].n_ct * st[k].n_pt;
        tiles += n;
        if (wide_step(st[k])) paired += n;
    }
    if (!chain && !h.issued && tiles >= kWideTiles && paired * kWideShare >= tiles) return launch_ns<T, kGatherMax, true, false>(h, st, sel, false, lc);
    // (the short block for the usual few steps: a third of the bytes to hand over)
    if constexpr (std::is_same<T, TraitsF32>::value) {
        bool any = false;
        for (int k = 0; k < h.n; ++k) any = any || stage_step(st[k]);
        if (!chain && !h.issued && any && tiles >= kStageTiles)
            return h.n <= 4 ? launch_ns<T, 4, false, true>(h, st, sel, false, lc) : launch_ns<T, kGatherMax, false, true>(h, st, sel, false, lc);
    }
    return h.n <= 4 ? launch_ns<T, 4, false, false>(h, st, sel, chain, lc) : launch_ns<T, kGatherMax, false, false>(h, st, sel, chain, lc);
}

}  // namespace

// How the tiles of a step lie (n_rows and the layer's shape are set).
void conv_gather_shape(bool first, GatherStep &a)
{
    auto rcp32 = [](int n) { return n > 1 ? (unsigned)((0x100000000ull + n - 1) / n) : 0u; };
    if (a.take == 1) { a.spt_log = 0; a.n_pt = a.n_cg = 1; return; }
    const int positions = a.n_rows * a.w_out;
    if (a.take == 2) { a.spt_log = 0; a.n_ct = a.n_cg = 1; a.n_pt = (positions * a.cells + kPoolCells - 1) / kPoolCells; a.ct_rcp = 0; return; }
    a.spt_log = streams_per_tile_log(positions, first);
    a.n_pt = (positions + (16 >> a.spt_log) - 1) / (16 >> a.spt_log);
    a.n_cg = a.n_ct;
    a.ct_rcp = rcp32(a.n_ct);
}

// The 1-D nets that go through units of this kernel from end to end, with pushes of all streams side by side.
bool cascade1d_eligible(int prec, const Geom *g, int n_layers, int max_seg_rows)
{
    if (prec != IDF_PREC_F32 || n_layers > kRowUnits || max_seg_rows > 16) return false;
    for (int l = 0; l < n_layers; ++l) {
        if (g[l].kind != IDF_CONV || g[l].w_in != 1 || g[l].w_out != 1 || g[l].k_w != 1) return false;
        if (g[l].c_in > 64 || g[l].c_out > 64 || g[l].k_h > 9 || g[l].s_h > 2 || g[l].k_h < g[l].s_h) return false;
        if (g[l].act != IDF_ACT_NONE && g[l].act != IDF_ACT_RELU) return false;
    }
    return true;
}

// Can a layer of a net of several kinds of layers go through this kernel, its ring holding ring_rows rows?  Strides are
// shifts here, divisions multiplications that have to be exact, and offsets into a stream's ring fit 31 bits; beyond
// 256 channels the generic kernels stay.
bool conv_gather_takes(int prec, const Geom &g, int ring_rows)
{
    const int vl = conv3x3_mfma_vl(prec), cells = (g.c_in + vl - 1) / vl;
    if (g.h_in < 1 || g.h_out < 1 || g.w_in > 4096 || g.c_in > 256 || g.c_out > 256) return false;
    if ((int64_t)ring_rows * g.w_in * cells * 16 > INT32_MAX || (int64_t)ring_rows * g.w_in >= 1 << 24) return false;
    if (g.kind == IDF_MAXPOOL) return true;
    auto shift = [](int s) { return s == 1 || s == 2 || s == 4; };
    if (!shift(g.s_h) || !shift(g.s_w) || g.k_h < g.s_h) return false;
    if (g.k_h > 32 || g.k_w > 32 || g.p_h >= g.k_h || g.p_w >= g.k_w) return false;
    // (rows of many positions: win_rcp is exact for any window of these sizes, at most 2,048 cells to a row of it and 65,539 in all)
    GatherStep a{};
    conv_gather_layer(prec, g, a);
    for (unsigned q = 0; a.flat && q < (unsigned)(g.k_h * cells); ++q)
        if (q * a.cells_rcp >> 16 != q / cells) return false;
    return true;
}

// What a step of a layer fetches from the caches to form `rows` rows of n_streams streams: a window and weights per tile.
double conv_gather_traffic(int prec, const Geom &g, int n_streams, int rows)
{
    GatherStep a{};
    conv_gather_layer(prec, g, a);
    return 2048.0 * a.n_ks * a.n_ct * ((double)n_streams * rows * g.w_out / 16);
}

// What a step needs to know of its layer whatever the rows.
void conv_gather_layer(int prec, const Geom &g, GatherStep &a)
{
    const int vl = conv3x3_mfma_vl(prec);
    auto log2i = [](int n) { int l = 0; while ((1 << l) < n) ++l; return l; };
    a.flat = g.w_in == 1 && g.w_out == 1 && g.k_w == 1 && g.p_w == 0;
    a.c_in = g.c_in; a.c_out = g.c_out; a.cells = (g.c_in + vl - 1) / vl;
    a.k_h = g.k_h; a.k_w = g.k_w; a.s_h_log = log2i(g.s_h); a.s_w_log = log2i(g.s_w); a.p_h = g.p_h; a.p_w = g.p_w;
    a.h_in = g.h_in > 0 ? g.h_in : INT32_MAX; a.w_in = g.w_in; a.h_out = g.h_out; a.w_out = g.w_out;
    a.act = g.act; a.shr = g.shr; a.clamp_hi = g.clamp_hi;
    a.take = g.kind == IDF_MAXPOOL ? 2 : 0;
    a.n_ct = (g.c_out + 15) / 16;
    a.n_ks = (g.k_h * g.k_w * a.cells + 3) / 4;
    a.cells_rcp = (unsigned)((65536 + a.cells - 1) / a.cells);
    const unsigned win_cells = (unsigned)(g.k_w * a.cells);
    a.win_rcp = win_cells > 1 ? (unsigned)((0x100000000ull + win_cells - 1) / win_cells) : 0u;
    a.wout_rcp = (unsigned)((0x100000000ull + g.w_out - 1) / g.w_out);
}

// Weights [k_h][k_w][c_in][c_out] -> [K-step][tile of 16 channels][lane][16 bytes], lane = 16 g + m holding cell 4 s + g of the
// K-step, counted (ky, kx, cell of channels), for channel m of the tile; zero padded.
size_t conv_gather_pack(int prec, const Geom &g, const void *w_khkwcico, void *out)
{
    const int vl = conv3x3_mfma_vl(prec), eb = 16 / vl, cells = (g.c_in + vl - 1) / vl, n_ct = (g.c_out + 15) / 16;
    const int n_ks = (g.k_h * g.k_w * cells + 3) / 4;
    const size_t bytes = (size_t)n_ks * n_ct * 1024;
    if (!out) return bytes;
    unsigned char *o = (unsigned char *)out;
    const unsigned char *src = (const unsigned char *)w_khkwcico;
    memset(o, 0, bytes);
    for (int tap = 0; tap < g.k_h * g.k_w; ++tap)
        for (int ci = 0; ci < g.c_in; ++ci) {
            const int q = tap * cells + ci / vl;
            for (int co = 0; co < g.c_out; ++co)
                memcpy(o + ((size_t)(q / 4) * n_ct + co / 16) * 1024 + (size_t)((q % 4) * 16 + co % 16) * 16 + (size_t)(ci % vl) * eb,
                       src + (((size_t)tap * g.c_in + ci) * g.c_out + co) * eb, eb);
        }
    return bytes;
}

hipError_t launch_ring_move(const RingMove &a, const LaunchCtx &lc)
{
    for (int k = 0; k < a.n_units; ++k)
        if (a.unit[k].keep * a.unit[k].row_cells > kMoveThreads) return hipErrorInvalidValue;      // (cascade1d_eligible: at most 9 rows of 16 cells)
    return launch(k_ring_move, dim3(a.n_units), dim3(kMoveThreads), 0, lc, a);
}

hipError_t launch_conv_gather(int prec, const GatherHead &h, const GatherStep *st, const StreamSel &sel, bool chain, const LaunchCtx &lc)
{
    if (h.n < 1 || h.n > kGatherMax) return hipErrorInvalidValue;
    switch (prec) {
    case IDF_PREC_F32: return launch_t<TraitsF32>(h, st, sel, chain, lc);
    case IDF_PREC_BF16: return launch_t<TraitsBf16>(h, st, sel, chain, lc);
    case IDF_PREC_I8: return launch_t<TraitsI8>(h, st, sel, chain, lc);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace idf
