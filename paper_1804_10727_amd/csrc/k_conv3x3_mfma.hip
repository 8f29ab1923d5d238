// Matrix-core event propagation for rows of a 3x3, stride 1, same-padded conv layer (bfloat16 events
// and weights -> float32 sums, int8 -> int32, or float32 throughout).
//
// The events of an arriving row are not delivered one row at a time into a retained row of c: they
// wait, in their own compact type, in a ring of the layer's input rows until the last row that an
// output row needs has arrived.  Then all events of its three input rows are delivered at once (the
// order of delivery does not matter to the sum, Sec. 3) and c lives in registers from its bias to
// its activation:
//     c[o][x][c_out] = bias + sum_{ky, kx, c_in} X[o - 1 + ky][x - 1 + kx][c_in] * W[ky][kx][c_in][c_out].
// A layer keeps K_h rows of events instead of K_h rows of four-byte sums, and a step reads rows and
// writes one row where it used to read two rows of c, add to three and write two back: on the
// VGG-style workload a launch of one row per stream moved 73 MB and took 20 us that way.
//
// A workgroup of four waves owns a stretch of positions and a group of output channels, for one output
// row or two.  Two rows share everything that is fetched: each weight serves both, and each of the
// two middle input rows is read from LDS once for both.
//   * The stretch of the input rows goes to LDS at once, a wave per row.  On the way every 16-byte cell
//     (channels of a position) that holds a non-zero sets a bit (a wave ballot, one word per row): K-steps
//     without events cost no matrix instruction, a stretch without events not even a weight fetch (zero
//     values are not events, Sec. 1).
//   * Operands are swapped: the matrix instruction's rows are output channels, its columns positions.
//     With the channels of a pair of tiles interleaved in the weight packing a lane then holds eight
//     neighbouring channels of one position, i.e. 16 bytes of a bfloat16 row: rows go straight from the
//     accumulators to memory, and the 2x2 max-pool is a maximum of two accumulators and one lane
//     exchange.
//   * The order of the sum is the same whatever a launch holds (K-step, tap row), so results do
//     not depend on how rows were grouped.
#include "idf.h"
#include "idf_kernels.h"
#include "mfma_tile.h"
#include <algorithm>
#include <cstddef>
#include <cstring>
#include <type_traits>

namespace idf {

namespace {

// A step's arguments, read where the launch put them (the kernel-argument segment): taken as an ordinary
// by-value argument, a block this large that is read in this many places is first copied to scratch memory.
typedef const __attribute__((address_space(4))) RowStep ArgStep;

constexpr int kWaves = 4, kThreads = 64 * kWaves;
// Where the waves of a workgroup add up their counters in LDS before one of them adds for all, and where each adds by itself.
// Additions to one place in memory go one after the other, and all waves of a step add to the same place per stream: what counts is how
// many workgroups a step has per stream -- with few there is little to wait for, and the trip to LDS costs more -- and whether other
// work covers the wait: with many streams, and earlier where tiles are wide and their waves four times as long, or events are few.
// us per image of 64 rows (int8: 112), by wave : by workgroup; in brackets the largest step's workgroups per stream.
//   bfloat16, 64 to 256 channels: 4 streams (14) 366 : 343 and, 8 rows per push (56), 157 : 107; (6) 355 : 348, (4) 342 : 333;
//     16 streams (14) 432 : 399, (6) 371 : 358, (4) 353 : 359; 24 streams (14) 485 : 476, 40 streams 511 : 510, 48 streams 564 : 570;
//     wide tiles (14 and 28) 16 streams 200 : 196, 20 streams 235 : 234, 24 streams 241 : 243, 64 streams 498 : 501
//   float32, 32 and 64 channels: (7) 8 streams 411 : 398, 32 streams 494 : 478, 48 streams 632 : 641; (2) 8 streams 384 : 392
//   int8, every other value an event, 64 and 128 channels: (14) 4 streams 547 : 543 and, two rows per push, 348 : 288; 16 streams 606 : 524;
//     32 to 128 channels, 8 rows per push (28), 24 streams 189 : 181; sparse events, 16 to 64 channels: (4) 16 streams 454 : 468;
//     8 rows per push (16), 3 streams 99 : 98, 24 streams 128 : 130
// (Kernels of their own: the branch alone, not taken, cost 256 small images 244 -> 248 us.)
constexpr int kTallyTiles = 5, kTallyStreams = 40, kTallyStreamsInt8 = 24, kTallyStreamsWide = 22;

// ---- rows of the caller: into the ring, and counted as the first layer's events --------------------
template <class T> __device__ __forceinline__ void take_row(ArgStep &a, const StreamSel &sel, const int tile, const int si)
{
    using ev_t = typename T::ev_t;
    const int tid = threadIdx.x, lane = tid & 63;
    const int stream = sel_stream(sel, si);
    const int y = a.y0 + tile, row_elems = a.w * a.c_in;
    const int slot = (a.slot0 + tile) % a.ring_rows;
    ev_t *ring = (ev_t *)a.in_ring + (int64_t)stream * a.in_stride + (int64_t)slot * row_elems;
    const ev_t *src = a.in_new ? (const ev_t *)a.in_new + (int64_t)(sel.pos0 + si) * a.new_stride + (int64_t)(y - a.y_new) * row_elems
                               : ring + a.x_lo * a.c_in;
    const bool save = a.in_new && y >= a.y_save;
    const int n = (a.x_hi - a.x_lo) * a.c_in;
    ev_t *dst = ring + a.x_lo * a.c_in;
    uint32_t ev = 0, tx = 0;
    if (a.cells > 0) {
        for (int i = tid; i < n / T::VL; i += kThreads) {
            const i32x4 v = reinterpret_cast<const i32x4 *>(src)[i];
            if (save) reinterpret_cast<i32x4 *>(dst)[i] = v;
            uint32_t k = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) k += T::nonzero((uint32_t)v[q]);
            ev += k; tx += k * taps_of(a.x_lo + i / a.cells, a.w);
        }
    } else {
        for (int i = tid; i < n; i += kThreads) {
            const ev_t v = src[i];
            if (save) dst[i] = v;
            if (T::ev_nonzero(v)) { ev += 1; tx += taps_of(a.x_lo + i / a.c_in, a.w); }
        }
    }
    if (!a.stats) return;
    ev = wave_sum(ev); tx = wave_sum(tx);
    if (lane == 0 && ev) {
        unsigned long long *d = a.stats + ((int64_t)stream * a.n_layers + a.layer) * 2;
        atomicAdd(d, (unsigned long long)ev);
        atomicAdd(d + 1, (unsigned long long)tx * (unsigned long long)(taps_of(y, a.h) * a.c_out));
    }
}

constexpr int kEvCap = 512;                      // events (stretch and halo) of a row the event path takes at most: 256 per 32 positions
// LDS of the event path behind the stretch: offsets and counts per position, the packed event list, the
// sums it hands to the accumulators, and the tile's share of the layer's weights.
constexpr size_t event_lds_bytes(int rows, int xt, int nc, int c_in) { return (size_t)(2 * (xt + 4) + kEvCap + rows * xt * nc + 3 * c_in * nc) * 4; }

// MC tiles of 16 channels x NP tiles of 16 positions x NR output rows per wave.  TAIL: windows may end within a K-step,
// in a float net: the weights behind are zero, but zero times infinity is not, so that what is read there has to be zero too.
template <class T, int MC, int NP, int NR, bool EV, bool TAIL, bool TALLY>
__device__ __forceinline__ void conv_rows(ArgStep &a, const StreamSel &sel, const int tile, const int si)
{
    using acc_t = typename T::acc_t; using st_t = typename T::st_t; using ev_t = typename T::ev_t;
    constexpr int VL = T::VL, EB = T::EB;
    constexpr int R = NR + 2;                      // input rows
    constexpr int NW = 3 * MC;                     // weight fragments of a K-step
    constexpr bool kFloat = std::is_same<st_t, float>::value;
    constexpr int kLoads = NP == 2 ? 18 : 9;       // cells each lane has in flight: a row of 32 positions (16) and halo x 32 cells at once
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ unsigned long long tally;           // what the waves have counted, and how many of them have
    __shared__ unsigned long long occ[kWaves];     // per input row, bit c: cell c holds an event somewhere in the stretch

    // Everything the loads need to know, asked for in one batch, and what the host can work out it has.  Left to first use the
    // arguments were a dozen scalar loads one after the other: from the arguments' arrival to the first request for a row 2,100 cycles,
    // now 1,000.  With weights asked for before the rows and the counters in one instruction (us per image, vgg-style net,
    // 64 streams / four out of step / 24 with 8 rows per push / f32 net: 2826 / 7030 / 663 / 285 before, 2576 / 5548 / 593 / 257 after).
    // What each is worth in the code as it stands, by taking it out: the batch nothing, now that little follows from the arguments
    // (2411 / 4587 / 539 / 250 -> 2427 / 4558 / 542 / 250), weights first 2466 / 4668 / 541 / 254, one instruction 2453 / 4666 / 567 / 252.
    const int n_rows = a.n_rows, y0 = a.y0, n_cg = a.n_cg, n_xt = a.n_xt, W = a.w, H = a.h, C_in = a.c_in, cells = a.cells, wc_log = a.wc_log;
    const int y_new = a.y_new, slot0 = a.slot0, ring_rows = a.ring_rows, nb = a.nb, n_ct = a.n_ct, co_g = a.co_g, n_ksteps = a.n_ksteps;
    const int C_out = a.c_out, stride = a.stride, row_pitch = a.row_pitch;     // (the last two: bytes in LDS from one position, and one row, to the next)
    const unsigned cg_rcp = a.cg_rcp, xt_rcp = a.xt_rcp, cells_rcp = a.cells_rcp, w_kstep = a.w_kstep, w_ky = a.w_ky;
    const int64_t in_stride = a.in_stride, new_stride = a.new_stride;
    const void *in_ring = a.in_ring, *in_new = a.in_new, *wfrag = a.wfrag, *bias = a.bias;
    const int sel_base = sel.base, pos0 = sel.pos0;
    asm volatile("" ::"s"(n_rows), "s"(y0), "s"(n_cg), "s"(n_xt), "s"(W), "s"(H), "s"(C_in), "s"(cells), "s"(wc_log), "s"(y_new), "s"(slot0), "s"(ring_rows),
                 "s"(nb), "s"(n_ct), "s"(co_g), "s"(cg_rcp), "s"(xt_rcp), "s"(cells_rcp), "s"(w_kstep), "s"(in_stride), "s"(new_stride), "s"(in_ring),
                 "s"(in_new), "s"(wfrag), "s"(bias), "s"(n_ksteps), "s"(sel_base));
    asm volatile("" ::"s"(w_ky), "s"(pos0), "s"(C_out), "s"(stride), "s"(row_pitch));

    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int m = lane & 15, g = lane >> 4;        // position within a tile; group of channels / of k
    const int stream = sel_base >= 0 ? sel_base + si : sel.ids[si];
    const int rest = (int)__umulhi((unsigned)tile, cg_rcp) + (n_cg == 1 ? tile : 0), cg = tile - rest * n_cg;
    const int rg = (int)__umulhi((unsigned)rest, xt_rcp) + (n_xt == 1 ? rest : 0), xt = rest - rg * n_xt;
    const int y = y0 + rg * NR;                    // first output row
    const int rows = n_rows - rg * NR < NR ? n_rows - rg * NR : NR;
    const int wc = wave & ((1 << wc_log) - 1), wp = wave >> wc_log;
    const int XT = (16 * NP * kWaves) >> wc_log;
    const int x0 = xt * XT;
    const int ct0 = ((cg << wc_log) + wc) * MC;    // first channel tile of this wave (16 channels: the only one; else tiles come in interleaved pairs)
    const int xw = x0 + wp * 16 * NP;              // first position of this wave
    const bool active = ct0 < n_ct && xw < W;
    // this lane's channels: co0 .. co0 + 4 * MC - 1
    const int co0 = (ct0 >> 1) * 32 + g * co_g + (MC == 1 ? (ct0 & 1) * 4 : 0);
    const bool co_ok = co0 < C_out;
    const bool small_c = cells == 0;

    // ---- weights -------------------------------------------------------------------------------------
    // [K-step][block of 32 channels][ky][tile of the pair][lane][16 bytes]  (one tile of channels: [K-step][ky][lane][16])
    constexpr int D = 3;                           // K-steps whose weights are on their way
    constexpr int D0 = NP == 2 ? 1 : D;            // of those, the ones asked for before the rows (as registers allow)
    const unsigned char *w_base[3];
    {
        const unsigned char *first = (const unsigned char *)wfrag + (active ? (ct0 >> 1) * 6144 + (MC == 1 ? (ct0 & 1) * 1024 : 0) : 0);
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) w_base[ky] = first + ky * w_ky;
    }
    uint32_t w_off = (uint32_t)lane * 16;
    int ks_left = n_ksteps;                        // K-steps whose weights have not been asked for
    auto fetch_w = [&](i32x4 (&w)[NW]) IDF_INLINE {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int mc = 0; mc < MC; ++mc) w[ky * MC + mc] = at4(reinterpret_cast<const i32x4 *>(w_base[ky]), w_off)[mc * 64];
        w_off += --ks_left > 0 ? w_kstep : 0u;     // past the end the last one is simply fetched again
    };
    acc_t acc[NR][MC][NP], start[MC];
    i32x4 w[D][NW];
#pragma unroll
    for (int d = 0; d < D0; ++d) {                 // (where rows lie is worked out while these are on their way)
        if (d > 0 && small_c) break;
        fetch_w(w[d]);
    }
#pragma unroll
    for (int mc = 0; mc < MC; ++mc) {
        start[mc] = acc_t{0, 0, 0, 0};
        if (bias) start[mc] = *reinterpret_cast<const acc_t *>((const st_t *)bias + (co_ok ? co0 : 0) + mc * 4);
    }

    // ---- input rows: wave r of the workgroup brings in input row r ------------------------------------
    auto row_there = [&](int r) IDF_INLINE { const int yi = y - 1 + r; return yi >= 0 && yi < H && r < rows + 2; };
    const bool there = wave < R && row_there(wave);
    const int row_bytes = W * C_in * EB;
    const unsigned char *my_row;                   // the same in every lane; a row that is not there: some row, whose values are dropped
    {
        const int yi = y - 1 + wave;
        int slot = slot0 + rg * NR + wave;
        slot = slot >= ring_rows ? slot - ring_rows : slot;
        const bool fresh = there && yi >= y_new;
        const int64_t at = fresh ? (int64_t)(pos0 + si) * new_stride : (int64_t)stream * in_stride;
        my_row = (const unsigned char *)(fresh ? in_new : in_ring) + at * EB + (int64_t)row_bytes * (there ? (fresh ? yi - y_new : slot) : 0);
    }
    // few channels: the stretch is kept as the windows the positions see, [row][position][3 * C_in values, padded to cells]
    const int wstride = stride;

    // ---- the stretch ----------------------------------------------------------------------------------
    if (!small_c) {
        // The whole stretch at once, in blocks of 64 cells (a position's cells are all its channels, so that a stretch lies in one
        // piece): everything this wave needs from memory is on its way together.  The registers it lands in are those of the
        // accumulators and fragments later.  A row in LDS is as long as whole blocks, so that no lane has to sit out.
        constexpr int kGroup = NP == 2 ? 9 : 3;    // blocks that are asked for without a look at how many there are
        static_assert(kLoads % kGroup == 0, "whole groups");
        const int first = (x0 - 1) * cells * 16 + lane * 16, last = row_bytes - 16;      // this lane's first cell, the row's last
        const bool edge = x0 == 0 || x0 + XT >= W;
        unsigned char *row = smem + wave * row_pitch;
        unsigned long long mask = 0;               // bit c: cell c holds an event somewhere in the stretch
        auto place = [&](int b) IDF_INLINE {       // of this lane's cell of block b
            const uint32_t i = (uint32_t)(b * 64 + lane);
            return reinterpret_cast<i32x4 *>(row + __umul24(__umul24(i, cells_rcp) >> 16, (uint32_t)(stride - cells * 16)) + i * 16);
        };
        if (there) {
            int any = 0;
            for (int b0 = 0; b0 < nb; b0 += kLoads) {
                i32x4 v[kLoads];
#pragma unroll
                for (int g0 = 0; g0 < kLoads; g0 += kGroup) {
                    if (b0 + g0 >= nb) break;
#pragma unroll
                    for (int b = g0; b < g0 + kGroup; ++b)
                        v[b] = *at4(reinterpret_cast<const i32x4 *>(my_row), (uint32_t)min(max(first + (b0 + b) * 1024, 0), last));
                }
#pragma unroll
                for (int b = 0; b < kLoads; ++b) {
                    if (b0 + b >= nb) break;
                    *place(b0 + b) = v[b];
                    const int o = T::or_of(v[b]);
                    any |= edge && (uint32_t)(first + (b0 + b) * 1024) > (uint32_t)last ? 0 : o;
                }
            }
            mask = __ballot(any != 0);
            if ((cells & (cells - 1)) == 0) {      // a lane has had one and the same cell throughout
                for (int c = 32; c >= cells; c >>= 1) mask |= mask >> c;
            } else {
                mask = mask ? ~0ull : 0ull;
            }
            // positions outside the row
            if (x0 == 0)
                for (int c = lane; c < cells; c += 64) *reinterpret_cast<i32x4 *>(row + c * 16) = i32x4{0, 0, 0, 0};
            if (x0 + XT >= W)
                for (int b = ((W - x0 + 1) * cells) >> 6; b < nb; ++b)
                    if (first + b * 1024 > last) *place(b) = i32x4{0, 0, 0, 0};
        } else if (wave < R) {
            for (int b = 0; b < nb; ++b) *place(b) = i32x4{0, 0, 0, 0};
        }
        if (lane == 0) occ[wave] = mask;
#pragma unroll
        for (int d = D0; d < D; ++d) fetch_w(w[d]);
        // a cell of zeros in the row's next position (there is one: 64 divides no such stretch)
        if (TAIL && (cells & 3) && wave < R && lane == 0) *reinterpret_cast<i32x4 *>(row + (XT + 2) * stride) = i32x4{0, 0, 0, 0};
    } else {
        // a lane gathers whole windows: three times C_in values next to each other in the row
        auto windows = [&](auto n_tag) IDF_INLINE {
            constexpr int C = decltype(n_tag)::value, WC = window_cells(C, VL, kFloat);
            if (wave >= R) return;
            for (int p = lane; p < XT; p += 64) {
                ev_t val[WC * VL];
#pragma unroll
                for (int k = 0; k < WC * VL; ++k) val[k] = 0;
                if (there) {
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) {
                        const int x = x0 - 1 + p + kx, xc = x < 0 ? 0 : (x >= W ? W - 1 : x);
#pragma unroll
                        for (int ci = 0; ci < C; ++ci) {
                            const ev_t v = *at4(reinterpret_cast<const ev_t *>(my_row), (uint32_t)((xc * C + ci) * EB));
                            val[kx * C + ci] = x == xc ? v : (ev_t)0;
                        }
                    }
                }
                i32x4 w[WC];
                __builtin_memcpy(w, val, sizeof(w));
#pragma unroll
                for (int k = 0; k < WC; ++k) *reinterpret_cast<i32x4 *>(smem + (wave * XT + p) * wstride + k * 16) = w[k];
            }
        };
        switch (C_in) {
        case 1: windows(std::integral_constant<int, 1>{}); break;
        case 2: windows(std::integral_constant<int, 2>{}); break;
        case 3: windows(std::integral_constant<int, 3>{}); break;
        default: windows(std::integral_constant<int, 4>{}); break;
        }
    }
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int mc = 0; mc < MC; ++mc)
#pragma unroll
            for (int np = 0; np < NP; ++np) acc[j][mc][np] = start[mc];
    // (likewise for what comes after the contraction)
    const int act = a.act, shr = a.shr, clamp_hi = a.clamp_hi, pool = a.pool, pool_from = a.pool_from, pool_emit = a.pool_emit, to_output = a.to_output;
    const int dst_slot0 = a.dst_slot0, dst_rows = a.dst_rows, layer = a.layer, pool_layer = a.pool_layer, next_layer = a.next_layer, next_c_out = a.next_c_out;
    const int n_layers = a.n_layers;
    const int64_t dst_stride = a.dst_stride;
    void *dst = a.dst;
    unsigned long long *stats = a.stats, *issued = a.issued;
    asm volatile("" ::"s"(act), "s"(shr), "s"(clamp_hi), "s"(pool), "s"(pool_from), "s"(pool_emit), "s"(to_output), "s"(dst_slot0), "s"(dst_rows), "s"(layer),
                 "s"(pool_layer), "s"(next_layer), "s"(next_c_out), "s"(n_layers), "s"(dst_stride), "s"(dst), "s"(stats), "s"(issued));
    if (TALLY && tid == 0) tally = 0;
    lds_barrier();
    uint32_t n_mfma = 0, n_done = 0;               // tiles of 16 x 16 x one K-step issued; K-steps issued

    // ---- sparse stretches: the event-list path ---------------------------------------------------------
    // Where a row's stretch (halo included) holds few events they are packed into a list -- counts per
    // position, an exclusive prefix sum, then (channel, value) words position by position -- and visited one by
    // one on the vector units: lanes = (position group, output channel), one weight word and one multiply-add
    // per event, output row and output channel.  The sums join the accumulators through LDS.
    uint32_t rows_done = 0;                        // input rows the list has taken care of (bit per row)
    if constexpr (EV && T::kEvents) {
        if (a.ev_limit > 0) {
            const int nc = 16 * MC << wc_log, pitch = a.row_pos;
            const size_t front = small_c ? (size_t)R * XT * wstride : (size_t)R * pitch * stride;
            int32_t *ev_cnt = reinterpret_cast<int32_t *>(smem + ((front + 15) & ~(size_t)15));
            int32_t *ev_off = ev_cnt + (XT + 4);
            uint32_t *ev_list = reinterpret_cast<uint32_t *>(ev_off + (XT + 4));
            int32_t *dsum = reinterpret_cast<int32_t *>(ev_list + kEvCap);          // [output row][position][channel]
            uint32_t *wlds = reinterpret_cast<uint32_t *>(dsum + NR * XT * nc);          // [kx][c_in][channel]
            const int cop = (C_out + 63) & ~63;
            {
                const uint32_t *wsrc = reinterpret_cast<const uint32_t *>(a.w_ev) + cg * nc;
                for (int i = tid; i < 3 * C_in * nc; i += kThreads) {
                    const int k = i / nc, c = i - k * nc;
                    wlds[i] = cg * nc + c < cop ? wsrc[(size_t)k * cop + c] : 0u;
                }
                for (int i = tid; i < NR * XT * nc; i += kThreads) dsum[i] = 0;
            }
            // value ci of stretch position p (p = 0: x0 - 1) of input row r
            auto value = [&](int r, int p, int ci) IDF_INLINE -> ev_t {
                if (!small_c) return reinterpret_cast<const ev_t *>(smem + (r * pitch + p) * stride)[ci];
                const int q = p == 0 ? 0 : p == XT + 1 ? XT - 1 : p - 1, kx = p == 0 ? 0 : p == XT + 1 ? 2 : 1;
                return reinterpret_cast<const ev_t *>(smem + (r * XT + q) * wstride)[kx * C_in + ci];
            };
            unsigned long long visits = 0;
            for (int r = 0; r < R; ++r) {
                if (!row_there(r)) { rows_done |= 1u << r; continue; }
                if (tid < XT + 2) {
                    int n = 0;
                    for (int ci = 0; ci < C_in; ++ci) n += T::ev_nonzero(value(r, tid, ci));
                    ev_cnt[tid] = n;
                }
                lds_barrier();
                if (tid <= XT + 2) {
                    int o = 0;
                    for (int q = 0; q < tid; ++q) o += ev_cnt[q];
                    ev_off[tid] = o;
                }
                lds_barrier();
                const int n_ev = uni(ev_off[XT + 2]);
                if (n_ev <= (XT > 32 ? 2 : 1) * a.ev_limit) {
                    rows_done |= 1u << r;
                    if (tid < XT + 2) {
                        int at = ev_off[tid];
                        for (int ci = 0; ci < C_in; ++ci) {
                            const ev_t v = value(r, tid, ci);
                            if (T::ev_nonzero(v)) ev_list[at++] = ((uint32_t)ci << 8) | (uint32_t)(uint8_t)v;
                        }
                    }
                    lds_barrier();
                    const int col = tid & (nc - 1), pg = tid / nc, n_pg = kThreads / nc;
                    for (int p = pg; p < XT && x0 + p < W; p += n_pg) {
                        const int i1 = ev_off[p + 1], i2 = ev_off[p + 2], i3 = ev_off[p + 3];
                        int32_t d[NR] = {};
                        for (int i = ev_off[p]; i < i3; ++i) {
                            const uint32_t e = ev_list[i];
                            const int kx = (i >= i1) + (i >= i2);
                            const uint32_t w = wlds[(kx * C_in + (int)(e >> 8)) * nc + col];
#pragma unroll
                            for (int j = 0; j < NR; ++j)
                                if (r - j >= 0 && r - j <= 2) d[j] += (int32_t)(int8_t)(e & 0xffu) * (int32_t)(int8_t)((w >> (8 * (r - j))) & 0xffu);
                        }
#pragma unroll
                        for (int j = 0; j < NR; ++j)
                            if (r - j >= 0 && r - j <= 2 && j < rows) {
                                dsum[(j * XT + p) * nc + col] += d[j];
                                if (col == 0) visits += (unsigned long long)(i3 - ev_off[p]);
                            }
                    }
                }
                lds_barrier();
                // a row that has been delivered reads as zero from here on
                if (!small_c && ((rows_done >> r) & 1u))
                    for (int i = tid; i < (XT + 2) * cells; i += kThreads)
                        *reinterpret_cast<i32x4 *>(smem + (r * pitch + i / cells) * stride + i % cells * 16) = i32x4{0, 0, 0, 0};
            }
            lds_barrier();
            if (a.issued && visits)
                atomicAdd(a.issued + (int64_t)stream * a.n_layers + a.layer, visits * (unsigned long long)nc);
            if (active) {
                const int cl = co0 - cg * nc;
#pragma unroll
                for (int j = 0; j < NR; ++j)
#pragma unroll
                    for (int mc = 0; mc < MC; ++mc)
#pragma unroll
                        for (int np = 0; np < NP; ++np)
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc[j][mc][np][i] += dsum[(j * XT + wp * 16 * NP + np * 16 + m) * nc + cl + mc * 4 + i];
            }
        }
    }

    // ---- contraction -------------------------------------------------------------------------------------
    // All matrix instructions of input row r's fragment of one K-step: tap row ky = r - j of output row j.
    auto deliver = [&](const i32x4 (&w)[NW], const i32x4 (&x)[NP], int r) IDF_INLINE {
#pragma unroll
        for (int e = 0; e < T::kInst; ++e)
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                const int ky = r - j;
                if (ky < 0 || ky > 2) continue;
#pragma unroll
                for (int mc = 0; mc < MC; ++mc)
#pragma unroll
                    for (int np = 0; np < NP; ++np) acc[j][mc][np] = T::mfma(w[ky * MC + mc], x[np], acc[j][mc][np], e);
            }
    };

    if (small_c) {
        // one K-step per tap row, always visited
        if (active) {
            const int wcells = window_cells(C_in, VL, kFloat);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (EV && ((rows_done >> r) & 1u)) continue;
                if (r >= rows + 2) continue;
                i32x4 x[NP];
#pragma unroll
                for (int np = 0; np < NP; ++np)
                    x[np] = *reinterpret_cast<const i32x4 *>(smem + (r * XT + wp * 16 * NP + np * 16 + m) * wstride + (kFloat || g < wcells ? g : wcells - 1) * 16);
                deliver(w[0], x, r);
                n_mfma += (uint32_t)(((r <= 2) + (NR == 2 && r >= 1 && rows == 2)) * MC * NP);
            }
        }
    }
    // K-step st holds cells 4 st .. 4 st + 3 of the window's 3 * cells, counted tap column by tap column.  Past the end the
    // weights are zero: the last one again, or (TAIL) a cell of zeros.
    unsigned long long mask = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        if (w < R && !(EV && ((rows_done >> w) & 1u))) mask |= occ[w];
    mask = (unsigned long long)(uint32_t)uni((int)(mask >> 32)) << 32 | (uint32_t)uni((int)mask);
    const bool by_cells = (cells & 3) == 0;    // every K-step lies in one tap column: its four cells have bits of their own
    const uint32_t pos = (uint32_t)((wp * 16 * NP + m) * stride);
    // With events in every K-step (bit 4 i of the mask's cells 4 i .. 4 i + 3) they go without a look at the mask: three K-steps' weights
    // and one K-step's cells ahead, and as few instructions in between as possible, which is what bounds a single wave (75 between
    // the six matrix instructions of a narrow K-step took 460 cycles, 35 take 210; wide tiles 885 -> 580, of which 384 are matrix
    // instructions.  Deeper requests alone, with the instructions as they were, gave nothing).
    // us per image before -> after: vgg-style net 2576 -> 2431, four streams out of step 5548 -> 5000, f32 net 257 -> 247.
    const unsigned long long some = (mask | mask >> 1 | mask >> 2 | mask >> 3) & 0x1111111111111111ull;
    const bool dense = by_cells && !small_c && (some << (64 - cells)) == 0x1111111111111111ull << (64 - cells);
    // (three blocks one after the other, of which one runs.  As branches of one another each would hold the first weights for
    // the others, 72 registers too many; the empty statement keeps them apart.)
    int n_dense = active && dense ? n_ksteps : 0, n_sparse = active && !small_c && !dense && mask ? n_ksteps : 0;
    asm volatile("" : "+s"(n_dense), "+s"(n_sparse));
    if (n_dense > 0) {
        i32x4 x[R][NP];
        uint32_t at = pos + (uint32_t)g * 16;
        auto read_row = [&](int r) IDF_INLINE {
#pragma unroll
            for (int np = 0; np < NP; ++np) x[r][np] = *reinterpret_cast<const i32x4 *>(smem + (at + (uint32_t)(r * row_pitch + np * 16 * stride)));
        };
#pragma unroll
        for (int r = 0; r < R; ++r) read_row(r);
        // A row's cells make room for those of the next K-step where they have been used.  The last round asks for nothing
        // more: the last weights once more, for the waits to count by, took the time of a request each and of registers that the
        // emission wants (us per image, vgg-style net, 64 streams / 24 streams, 8 rows per push: 2468 -> 2381, 598 -> 568).
        int left = n_dense, col = cells >> 2;
        const uint32_t over = (uint32_t)(stride - cells * 16);
        auto advance = [&]() IDF_INLINE {
            at += 64u;
            if (--col == 0) { at += over; col = cells >> 2; }
        };
#pragma unroll 1
        for (; left > D; left -= D) {          // (three tap columns: whole rounds)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                advance();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    deliver(w[d], x[r], r);
                    read_row(r);
                    __builtin_amdgcn_sched_barrier(0);
                }
                fetch_w(w[d]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d < D - 1) advance();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                deliver(w[d], x[r], r);
                if (d < D - 1) read_row(r);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        n_done = n_dense;
    }
    if (n_sparse > 0) {
        auto kstep = [&](const i32x4 (&wv)[NW], int st) IDF_INLINE {
            int q = 4 * st + g;
            const bool past = TAIL && q >= 3 * cells;
            q = q < 3 * cells ? q : 3 * cells - 1;
            const int kx = (q >= cells) + (q >= 2 * cells);
            const uint32_t off = past ? (uint32_t)((XT + 2) * stride) : pos + (uint32_t)(kx * stride + (q - kx * cells) * 16);
            const uint32_t np_pitch = past ? 0u : (uint32_t)(16 * stride);
            i32x4 x[R][NP];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int np = 0; np < NP; ++np) x[r][np] = *reinterpret_cast<const i32x4 *>(smem + off + r * row_pitch + np * np_pitch);
#pragma unroll
            for (int r = 0; r < R; ++r) deliver(wv, x[r], r);
            ++n_done;
        };
        unsigned long long rest = mask;
        int col_left = by_cells ? cells >> 2 : 1 << 30;       // K-steps to the end of the tap column
        auto live = [&]() IDF_INLINE { return by_cells ? ((uint32_t)rest & 0xfu) != 0 : true; };
        auto next = [&]() IDF_INLINE {
            rest >>= 4;
            if (--col_left == 0) { rest = mask; col_left = cells >> 2; }
        };
        // (the first two have their weights; what the prologue asked for beyond them is asked for again)
        if (D > 2) { ks_left = n_ksteps > 2 ? n_ksteps - 2 : 0; w_off = (uint32_t)lane * 16 + (uint32_t)(n_ksteps > 2 ? 2 : n_ksteps - 1) * w_kstep; }
#pragma unroll 1
        for (int st = 0;; st += 2) {
            if (live()) kstep(w[0], st);
            if (st + 1 >= n_ksteps) break;
            fetch_w(w[0]);
            next();
            __builtin_amdgcn_sched_barrier(0);  // K-steps stay apart: nothing of a later one is held in registers early
            if (live()) kstep(w[1], st + 1);
            if (st + 2 >= n_ksteps) break;
            fetch_w(w[1]);
            next();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (!active) return;

    // ---- the rows are final: activate, emit, count ---------------------------------------------------------
    // (a lane's place is worked out again rather than held in registers through the contraction: the empty statement hides that it
    // is the same value)
    int id = tid;
    asm volatile("" : "+v"(id));
    const int me = id & 15, co1 = (ct0 >> 1) * 32 + (id >> 4 & 3) * co_g + (MC == 1 ? (ct0 & 1) * 4 : 0);
    constexpr int NV = 4 * MC;                     // neighbouring channels a lane holds
    uint32_t next = 0, pooled = 0;                 // events for the next layer (high half: their taps), events the pool receives
    auto emit = [&](const uint32_t (&e)[MC * EB], int row_w, int x, int slot) IDF_INLINE {
        unsigned char *d = (unsigned char *)dst + ((int64_t)stream * dst_stride + (int64_t)slot * row_w * C_out) * EB;
        const uint32_t off = (uint32_t)((x * C_out + co1) * EB);
        // bfloat16 rows go through the L2 to memory at once: left there they are written back behind the last workgroup, and the next launch
        // waits for it (us per image, vgg-style net, 64 streams / four out of step / 24 with 8 rows per push: 2382 -> 2314, 4565 -> 4426,
        // 528 -> 520; past both caches, `nt`, 2455, 4688, 560.  float32 rows, half of a line per store, 248 -> 250; rows of the output,
        // which are larger, 2314 -> 2402; what the gathering kernel emits the same either way).  In launches of 2,500 to 7,500 positions either
        // way is ahead by up to 1 %, with no order in width or streams: 29 streams of 57 x 130 406 -> 410, 24 of 48 x 200 357 -> 361, 28 of 48 x 224
        // 388 -> 384, 43 of 73 x 176 683 -> 678; below and above it is this one, 12 of 48 x 224 292 -> 290, 56 of 48 x 224 497 -> 483.  Asking whether a
        // launch of narrow tiles has 3,600 positions or fewer costs what it gains: 24 of 48 x 200 1.004 of the time without -> 0.997, 28 of 48 x 224
        // 0.985 -> 0.998, 32 of 48 x 128 with two rows 0.992 -> 1.013.
        // The s_nop: gfx950 wants two wait states between a store of more than eight bytes and a vector instruction that writes its registers,
        // which the compiler sees to for its own stores only.
        if constexpr (MC * EB == 1) *at4(reinterpret_cast<uint32_t *>(d), off) = e[0];
        else if constexpr (MC * EB == 2) {
            const i32x2 v{(int)e[0], (int)e[1]};
            if constexpr (EB == 2) asm volatile("global_store_dwordx2 %0, %1, %2 sc1" ::"v"(off), "v"(v), "s"(d) : "memory");
            else *at4(reinterpret_cast<i32x2 *>(d), off) = v;
        } else {
#pragma unroll
            for (int q = 0; q < MC * EB / 4; ++q) {
                const i32x4 v{(int)e[4 * q], (int)e[4 * q + 1], (int)e[4 * q + 2], (int)e[4 * q + 3]};
                if constexpr (EB == 2) asm volatile("global_store_dwordx4 %0, %1, %2 sc1\n\ts_nop 1" ::"v"(off + q * 16), "v"(v), "s"(d) : "memory");
                else *at4(reinterpret_cast<i32x4 *>(d), off + q * 16) = v;
            }
        }
    };
    auto emit_out = [&](const st_t (&v)[NV], int row_w, int x, int slot) IDF_INLINE {        // last layer: 4-byte values, not rounded to the event type
        st_t *d = (st_t *)dst + (int64_t)stream * dst_stride + (int64_t)slot * row_w * C_out;
#pragma unroll
        for (int q = 0; q < MC; ++q)
            *at4(reinterpret_cast<acc_t *>(d), (uint32_t)((x * C_out + co1 + q * 4) * 4)) = acc_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    };
    const FloatBounds bounds(act == IDF_ACT_NONE);
    auto activated = [&](st_t c) IDF_INLINE {
        if constexpr (kFloat) return bounds(c);
        else return T::activate(c, act, shr, clamp_hi);
    };
    auto count = [&](const uint32_t (&e)[MC * EB]) IDF_INLINE {
        uint32_t n = 0;
#pragma unroll
        for (int q = 0; q < MC * EB; ++q) n += (uint32_t)T::nonzero(e[q]);
        return n;
    };
    auto slot_of = [&](int i) IDF_INLINE { int s = dst_slot0 + i; return s >= dst_rows ? s - dst_rows : s; };
#pragma unroll
    for (int np = 0; np < NP; ++np) {
        const int x = xw + np * 16 + me;
        const bool ok = x < W && co1 < C_out;
        if (!pool) {
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                if (j >= rows) break;
                st_t v[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) v[q] = activated(acc[j][q >> 2][np][q & 3]);
                if (!ok) continue;
                if (to_output) {
                    emit_out(v, W, x, slot_of(rg * NR + j));
                } else {
                    uint32_t e[MC * EB];
#pragma unroll
                    for (int q = 0; q < MC; ++q) T::pack4(v + 4 * q, e + q * EB);
                    emit(e, W, x, slot_of(rg * NR + j));
                    if (next_layer >= 0) {
                        const uint32_t n = count(e);
                        next += n + ((n * (uint32_t)(taps_of(x, W) * taps_of(y + j, H))) << 16);
                    }
                }
            }
        } else {
            // 2x2 max over the two rows and the neighbouring position; rounding does not change the order of values
            st_t v[NV];
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                if (j >= rows) break;
                st_t u[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) u[q] = activated(acc[j][q >> 2][np][q & 3]);
                if (y + j >= pool_from && ok) {
                    uint32_t e[MC * EB];
#pragma unroll
                    for (int q = 0; q < MC; ++q) T::pack4(u + 4 * q, e + q * EB);
                    pooled += count(e);
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) v[q] = j == 0 ? u[q] : (u[q] > v[q] ? u[q] : v[q]);
            }
            if (NR == 2 && rows == 2 && pool_emit) {
#pragma unroll
                for (int q = 0; q < NV; ++q) { const st_t o = neighbour(v[q]); v[q] = o > v[q] ? o : v[q]; }
                const int Wp = W >> 1, xp = x >> 1, yp = y >> 1;
                if (ok && !(me & 1) && xp < Wp) {
                    if (to_output) {
                        // (a pool as the last layer: float32 nets only, whose events are the values)
                        emit_out(v, Wp, xp, slot_of(rg));
                    } else {
                        uint32_t e[MC * EB];
#pragma unroll
                        for (int q = 0; q < MC; ++q) T::pack4(v + 4 * q, e + q * EB);
                        emit(e, Wp, xp, slot_of(rg));
                        if (next_layer >= 0) {
                            const uint32_t n = count(e);
                            next += n + ((n * (uint32_t)(taps_of(xp, Wp) * taps_of(yp, H >> 1))) << 16);
                        }
                    }
                }
            }
        }
    }
    if (stats) {
        // (three lanes, one instruction: events of the next layer, the multiply-adds they stand for, events of the pool)
        next = wave_sum(next);
        pooled = wave_sum(pooled);
        uint32_t events = next & 0xffffu, taps = next >> 16;
        bool last = true;
        if constexpr (TALLY) {                     // the last of the workgroup's waves adds for all
            const int n_wc = min(1 << wc_log, (n_ct - (cg << wc_log) * MC + MC - 1) / MC), n_wp = min(kWaves >> wc_log, (W - x0 + 16 * NP - 1) / (16 * NP));
            const uint64_t mine = (uint64_t)events | (uint64_t)taps << 14 | (uint64_t)pooled << 31 | 1ull << 45;     // (at most 8,192 events, nine taps each)
            uint64_t before = 0;
            if ((id & 63) == 0)
                asm volatile("ds_add_rtn_u64 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)"
                             : "=v"(before) : "v"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned long long *)&tally), "v"(mine) : "memory");
            const uint64_t all = mine + ((uint64_t)(uint32_t)uni((int)(before >> 32)) << 32 | (uint32_t)uni((int)before));
            last = (int)(all >> 45) == n_wc * n_wp;
            events = (uint32_t)all & 0x3fffu; taps = (uint32_t)(all >> 14) & 0x1ffffu; pooled = (uint32_t)(all >> 31) & 0x3fffu;
        }
        const uint64_t add = (id & 63) == 0 ? events : (id & 63) == 1 ? (uint64_t)taps * (uint32_t)next_c_out : pooled;
        if (last && (id & 63) < 3 && add)
            atomicAdd(stats + ((int64_t)stream * n_layers + ((id & 63) == 2 ? pool_layer : next_layer)) * 2 + ((id & 63) == 1), (unsigned long long)add);
    }
    // what the matrix instructions of this wave multiplied, zeros inside a live K-step included
    n_mfma += n_done * (uint32_t)(3 * rows * MC * NP);
    if (issued && (id & 63) == 0 && n_mfma)
        atomicAdd(issued + (int64_t)stream * n_layers + layer, (unsigned long long)n_mfma * (256ull * 4 * VL));
}

// Several layers' steps in one launch (each on rows that were complete before the launch).  The grid is
// (stream, tile, step): a workgroup knows its step from its own index, so its arguments arrive in one
// round of scalar loads.  Steps with fewer tiles than the launch's largest leave workgroups that return
// at once.  In dispatch order the streams of a tile lie side by side, then the tiles of a step, then the
// steps with the deepest (longest) first.  Consecutive workgroups go to the eight XCDs in turn: with a
// multiple of eight streams a stream always meets the same XCD, so its rows stay in one L2 from the layer
// that emits them to the layer that reads them.
template <class T, bool EV, bool WIDE, bool TAIL, bool TALLY>
__global__ void __launch_bounds__(kThreads, 3) k_conv3x3_mfma_rows(const RowBatch b, const StreamSel sel)
{
    (void)b;                                      // the first argument: it begins the segment
    const __attribute__((address_space(4))) char *args = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
    ArgStep &a = *((ArgStep *)(args + offsetof(RowBatch, st)) + blockIdx.z);
    const int tile = blockIdx.y, si = blockIdx.x;
    // (by every workgroup; us per pass, none / the first 256 / all: vgg-style net 3006 / 2925 / 2850, four streams out of step
    //  7256 / 7150 / 7030, float32 net 300 / 292 / 284)
    request_arguments<sizeof(RowStep), kWaves>(&a, args + sizeof(RowBatch));          // (the streams behind)
    const int tiles = a.tiles, form = a.form;
    asm volatile("" ::"s"(tiles), "s"(form));
    if (tile >= tiles) return;
    switch (form) {
    case kRowTake: take_row<T>(a, sel, tile, si); break;
    case kRowSmall1: conv_rows<T, 1, 1, 1, EV, TAIL, TALLY>(a, sel, tile, si); break;
    case kRowSmall2: conv_rows<T, 1, 1, 2, EV, TAIL, TALLY>(a, sel, tile, si); break;
    case kRowWide2: if constexpr (WIDE) conv_rows<T, 2, 2, 2, false, TAIL, TALLY>(a, sel, tile, si); break;
    default: break;
    }
}

int form_np(int form) { return form == kRowWide2 ? 2 : 1; }
int form_rows(int form) { return form == kRowSmall1 ? 1 : 2; }

size_t step_lds(const RowStep &a)
{
    if (a.form == kRowTake) return 0;
    const int rows = form_rows(a.form) + 2;
    return (size_t)rows * a.row_pitch;
}

constexpr int kRowLds = 160 * 1024 - 256;         // of a workgroup at most, beside what the kernel declares

template <class T> hipError_t launch_rows(int prec, const RowBatch &b, const StreamSel &sel, const LaunchCtx &lc)
{
    size_t lds = 0;
    int tiles = 0, counting = 0;                   // workgroups per stream: of the largest step, and of the largest whose waves count
    bool events = false, wide = false, tail = false;
    for (int k = 0; k < b.n; ++k) {
        const RowStep &a = b.st[k];
        tiles = std::max(tiles, a.tiles);
        if (a.form != kRowTake && (a.pool || a.next_layer >= 0)) counting = std::max(counting, a.tiles);
        wide = wide || a.form == kRowWide2;
        tail = tail || (prec != IDF_PREC_I8 && a.form != kRowTake && (a.cells & 3));
        size_t need = step_lds(a);
        if (a.ev_limit > 0) {
            events = true;
            need = ((need + 15) & ~(size_t)15) + event_lds_bytes(form_rows(a.form), (16 * kWaves) >> a.wc_log, 16 << a.wc_log, a.c_in);
        }
        lds = std::max(lds, need);
    }
    if (b.n < 1 || tiles < 1 || tiles > kRowTilesMax || lds > kRowLds) return hipErrorInvalidValue;      // tiles are the grid's y extent
    const dim3 grid(sel.n, tiles, b.n), block(kThreads);
    auto go = [&](auto kernel) {
        const hipError_t e = allow_lds<kRowLds>(kernel);
        return e != hipSuccess ? e : launch(kernel.entry, grid, block, lds, lc, b, sel);
    };
    constexpr bool kF32 = std::is_same<T, TraitsF32>::value;
    if (wide && (kF32 || events)) return hipErrorInvalidValue;
    auto pick = [&](auto tally_tag) {
        constexpr bool TALLY = decltype(tally_tag)::value;
        if constexpr (T::kEvents) {
            if (events) return go(Kernel<k_conv3x3_mfma_rows<T, true, false, false, TALLY>>{});
        } else if (tail) {
            // (a kernel of its own: where the kernel below had a few instructions for it -- a branch, a comparison per K-step, or
            // unused loops beside the others -- nets without such layers took 1 to 2 % longer, float32 283 -> 288 us per image)
            return wide ? go(Kernel<k_conv3x3_mfma_rows<T, false, !kF32, true, TALLY>>{}) : go(Kernel<k_conv3x3_mfma_rows<T, false, false, true, TALLY>>{});
        }
        return wide ? go(Kernel<k_conv3x3_mfma_rows<T, false, !kF32, false, TALLY>>{}) : go(Kernel<k_conv3x3_mfma_rows<T, false, false, false, TALLY>>{});
    };
    const bool by_group = counting >= kTallyTiles && sel.n < (wide ? kTallyStreamsWide : T::kEvents ? kTallyStreamsInt8 : kTallyStreams);
    return by_group ? pick(std::true_type{}) : pick(std::false_type{});
}

}  // namespace

// Elements of the event type per 16-byte cell.
int conv3x3_mfma_vl(int prec) { return prec == IDF_PREC_F32 ? 4 : prec == IDF_PREC_BF16 ? 8 : 16; }

bool conv3x3_mfma_eligible(int prec, const Geom &g)
{
    if (prec != IDF_PREC_BF16 && prec != IDF_PREC_I8 && prec != IDF_PREC_F32) return false;
    const int vl = conv3x3_mfma_vl(prec);
    if (g.kind != IDF_CONV || g.k_h != 3 || g.k_w != 3 || g.s_h != 1 || g.s_w != 1 || g.p_h != 1 || g.p_w != 1) return false;
    if (g.h_in < 2 || g.w_in < 2) return false;
    if ((g.c_in % vl != 0 && g.c_in > 4) || g.c_out % 16 != 0) return false;
    const int steps = (3 * g.c_in + 2 * vl - 1) / (2 * vl);
    if (steps > 64 || g.c_in / vl > 64) return false;
    return true;
}

// K-steps (of four cells) per tap row.
static int row_ksteps(int prec, const Geom &g)
{
    const int vl = conv3x3_mfma_vl(prec);
    if (g.c_in % vl != 0 || g.c_in < vl) return 1;
    return (3 * (g.c_in / vl) + 3) / 4;
}

// Waves of a step in tiles of 32 positions x 32 channels (0: it cannot have such).  float32 stays narrow, its matrix instructions being
// sixteen times longer.  So do all steps next to one on the event path: one kernel with both wants more registers than three waves per
// SIMD leave (20 bytes of scratch).
int64_t conv3x3_mfma_wide_waves(int prec, const Geom &g, int n_streams, const RowStep &a)
{
    if (prec == IDF_PREC_F32 || a.ev_limit != 0 || a.n_rows < 2 || g.c_out <= 16) return 0;
    return (int64_t)n_streams * ((g.w_out + 31) / 32) * ((g.c_out + 31) / 32) * ((a.n_rows + 1) / 2);
}

// Wide tiles use each weight fragment and each cell twice as often.  A step of its own has them where they give every SIMD most of a
// wave; any but the smallest where the launch's steps together fill the chip with them, since weights on their way to the registers are
// what bounds narrow ones then (42 bytes per clock and CU).  us per image, bfloat16, 64 to 256 channels, by step alone : with the launch
// counted; streams of 96 x 224, rows per push:
//   24 of 1 row 720 : 723, 32 798 : 778, 40 954 : 927, 48 957 : 911; 24 of 2 rows 554 : 513, 32 679 : 552; 12 of 4 296 : 295, 16 355 : 330,
//   24 441 : 360; 8 of 8 195 : 185, 12 259 : 232, 16 301 : 260, 24 332 : 310; 60 of 96 x 100, 1 and 2 rows 792 : 780, 655 : 558.
//   From 1,280 waves on in place of 1,400: 64 of 96 x 64, 2 rows, 433 : 436 : 478.  From 1,152 on: 12 of 4 rows 282 : 298.  From 1,792 on:
//   24 of 2 rows 524 : 523, 40 of 1 row 910 : 889.  All steps of 192 and more, whatever the launch: 16 of 2 rows 402 : 474, 24 of 1 705 : 771.
//   Steps of 256 and more in place of 192: 12 of 4 rows 303.  int8 the same either way (64 of 96 x 150, 4 rows, 197 : 195).
constexpr int kWideAlone = 768, kWideLeast = 192;

// Shape of a step of n_rows output rows for n_streams streams: which tiles a wave takes, how the waves of a
// workgroup lie, and the numbers that follow from that.
void conv3x3_mfma_shape(int prec, const Geom &g, int n_streams, bool narrow, int64_t launch_waves, RowStep &a)
{
    const int vl = conv3x3_mfma_vl(prec);
    a.cells = g.c_in % vl == 0 && g.c_in >= vl ? g.c_in / vl : 0;
    const int n_ct = g.c_out == 16 ? 1 : 2 * ((g.c_out + 31) / 32);
    const int64_t waves = narrow ? 0 : conv3x3_mfma_wide_waves(prec, g, n_streams, a);
    const bool wide = waves >= kWideAlone || (waves >= kWideLeast && launch_waves >= kWideLaunch);
    auto waves_log = [&](int tiles) { return tiles >= 4 ? 2 : tiles >= 2 ? 1 : 0; };
    a.wc_log = waves_log(wide ? n_ct / 2 : n_ct);
    // A stretch short enough for two workgroups to share a CU's LDS.  The waves it does not need for positions take channels; where
    // there are none left for them they load rows and leave, which is still better than one workgroup per CU (bfloat16, 224
    // positions, 8 rows per push: 64 -> 32 channels 555 us per image against 775, 256 -> 64 543 against 605).
    while (a.wc_log < 2 && (((wide ? 128 : 64) >> a.wc_log) + 2) * cell_stride(std::max(a.cells, 1)) * 4 * 16 > 76 * 1024) ++a.wc_log;
    a.form = wide ? kRowWide2 : a.n_rows >= 2 ? kRowSmall2 : kRowSmall1;
    const int mc = a.form == kRowWide2 ? 2 : 1, xt = (16 * form_np(a.form) * kWaves) >> a.wc_log;
    auto rcp32 = [](int n) { return n > 1 ? (unsigned)((0x100000000ull + n - 1) / n) : 0u; };
    a.n_xt = (g.w_out + xt - 1) / xt;
    a.n_cg = (n_ct + (mc << a.wc_log) - 1) / (mc << a.wc_log);
    a.xt_rcp = rcp32(a.n_xt); a.cg_rcp = rcp32(a.n_cg);
    a.tiles = (a.n_rows + form_rows(a.form) - 1) / form_rows(a.form) * a.n_xt * a.n_cg;
    const int cells = std::max(a.cells, 1);
    a.nb = ((xt + 2) * cells + 63) / 64;
    a.row_pos = (a.nb * 64 + cells - 1) / cells;
    a.cells_rcp = (unsigned)((65536 + cells - 1) / cells);
    a.stride = cell_stride(a.cells ? cells : window_cells(g.c_in, vl, prec != IDF_PREC_I8)) * 16; a.row_pitch = (a.cells ? a.row_pos : xt) * a.stride;
    const bool single = g.c_out == 16;
    a.n_ct = n_ct; a.co_g = single ? 4 : 8;
    a.n_ksteps = a.cells ? (3 * a.cells + 3) / 4 : 1;
    a.w_kstep = single ? 3 * 1024 : (unsigned)((g.c_out + 31) / 32) * 6144; a.w_ky = single ? 1024 : 2048;
}

bool conv3x3_mfma_split(RowStep &first, RowStep &rest)
{
    const int pairs = first.form == kRowTake ? 1 : form_rows(first.form), per = first.form == kRowTake ? 1 : first.n_xt * first.n_cg;
    const int n = kRowTilesMax / per * pairs;
    if (n < 1 || n >= first.n_rows) return false;
    rest = first;
    first.n_rows = n;
    first.tiles = n / pairs * per;
    rest.n_rows -= n; rest.y0 += n;
    rest.tiles = (rest.n_rows + pairs - 1) / pairs * per;
    rest.slot0 = (rest.slot0 + n) % rest.ring_rows;
    if (first.form != kRowTake) rest.dst_slot0 = (rest.dst_slot0 + (first.pool ? n / 2 : n)) % rest.dst_rows;
    return true;
}

// Weights [k_h][k_w][c_in][c_out] -> fragment order, zero padded to whole K-steps and channel pairs:
//   [K-step][block of 32 channels][ky][tile t of 2][lane][16 bytes], lane = 16 g + m holding cell 4 s + g of the
//   K-step for row m of the tile, which is channel 32 * block + (m / 4) * 8 + t * 4 + m % 4;
//   16 output channels: [K-step][ky][lane][16 bytes], row m = channel m.
// K-steps run over the cells kx * (cells per position) + c; with one to four input channels there is one K-step whose
// elements are k = kx * c_in + ci.
size_t conv3x3_mfma_pack(int prec, const Geom &g, const void *w_khkwcico, void *out)
{
    const int vl = conv3x3_mfma_vl(prec), eb = 16 / vl;
    const int ksteps = row_ksteps(prec, g), n_blk = (g.c_out + 31) / 32;
    const bool single = g.c_out == 16;
    const size_t per_step = single ? 3 * 1024 : (size_t)n_blk * 6144, frag_bytes = per_step * ksteps;
    const int cop = (g.c_out + 63) / 64 * 64;
    // int8: behind the fragments the same weights for the event path, [kx][c_in][cop] words holding the taps ky = 0, 1, 2 of
    // (kx, c_in, c_out) in their three low bytes
    const size_t bytes = frag_bytes + (prec == IDF_PREC_I8 ? (size_t)3 * g.c_in * cop * 4 : 0);
    if (!out) return bytes;
    unsigned char *o = (unsigned char *)out;
    const unsigned char *src = (const unsigned char *)w_khkwcico;
    memset(o, 0, bytes);
    const int cells = g.c_in % vl == 0 && g.c_in >= vl ? g.c_in / vl : 0;
    for (int ky = 0; ky < 3; ++ky)
        for (int kx = 0; kx < 3; ++kx)
            for (int ci = 0; ci < g.c_in; ++ci) {
                int step, grp, elem;
                if (cells == 0) {
                    const int k = kx * g.c_in + ci;
                    step = 0; grp = k / vl; elem = k % vl;
                } else {
                    const int q = kx * cells + ci / vl;
                    step = q / 4; grp = q % 4; elem = ci % vl;
                }
                for (int co = 0; co < g.c_out; ++co) {
                    const size_t s_idx = (((size_t)ky * 3 + kx) * g.c_in + ci) * g.c_out + co;
                    size_t d;
                    if (single) {
                        d = step * per_step + (size_t)ky * 1024 + (size_t)(grp * 16 + co) * 16;
                    } else {
                        const int in = co % 32, t = in % 8 / 4, m = in / 8 * 4 + in % 4;
                        d = step * per_step + (size_t)(co / 32) * 6144 + (size_t)(ky * 2 + t) * 1024 + (size_t)(grp * 16 + m) * 16;
                    }
                    if (eb == 4) memcpy(o + d + (size_t)elem * 4, src + s_idx * 4, 4);
                    else if (eb == 2) memcpy(o + d + (size_t)elem * 2, src + s_idx * 2, 2);
                    else o[d + (size_t)elem] = src[s_idx];
                    if (prec == IDF_PREC_I8) o[frag_bytes + (((size_t)kx * g.c_in + ci) * cop + co) * 4 + ky] = src[s_idx];
                }
            }
    return bytes;
}

size_t conv3x3_mfma_event_weights(int prec, const Geom &g)
{
    if (prec != IDF_PREC_I8) return 0;
    return (g.c_out == 16 ? 3 * 1024 : (size_t)((g.c_out + 31) / 32) * 6144) * row_ksteps(prec, g);
}

int conv3x3_mfma_event_cap() { return kEvCap / 2; }

hipError_t launch_conv3x3_mfma_rows(int prec, const RowBatch &b, const StreamSel &sel, const LaunchCtx &lc)
{
    if (prec == IDF_PREC_F32) return launch_rows<TraitsF32>(prec, b, sel, lc);
    if (prec == IDF_PREC_BF16) return launch_rows<TraitsBf16>(prec, b, sel, lc);
    if (prec == IDF_PREC_I8) return launch_rows<TraitsI8>(prec, b, sel, lc);
    return hipErrorInvalidValue;
}

}  // namespace idf
