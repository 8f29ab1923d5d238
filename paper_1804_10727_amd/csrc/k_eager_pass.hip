// Eager emission of one segment through a whole net of 3x3 / stride 1 / same-padded conv layers and 2x2
// max-pools in one launch: a workgroup takes one stream from the pushed rows to the output, or, where pushes follow one another
// without a read, through one stage of a few layers while others take the pushes before it through the stages behind (eager_stages in
// idf_lib.hip has the rule and both sides of it; int8, eight streams of 112 x 112: 3195 -> 1126 us per image, and with several workgroups
// to a stage 776; float32, 256 streams of 32 x 32: 1028 -> 952).
//
// A segment's events are a band of a few rows per layer, so layer by layer the work is small and the time
// went into launches, into memory round trips between them and into finding the events: the 8 conv layers
// of the int8 network at 8 streams of 112 x 112 took 8 launches of 20 us.  Here
//   * the differences announced by a layer stay in LDS for the next one, which multiplies all of them on
//     the matrix cores (float32 as 16x16x4, int8 as 16x16x64: differences of values in 0..127 are int8
//     again, and exact).  A wave takes 16 channels x 16 positions of four rows of the layer (the first
//     of them even, so that no window of a pool is divided), and of those only what the band reaches;
//   * what a cell had announced is f of the state it had, so only the state is read; a pool's windows are
//     maxima of two rows in registers and one exchange of lanes;
//   * between layers there is one barrier over LDS; the stores of state and announced values are not waited for.
// What bounds it is the chain: every layer is a memory round trip for its weights, a few dozen matrix
// instructions and some five hundred others per wave, one after the other.  Hence sixteen waves with small shares
// (eight waves with all the rows of a band each took 1.3 times as long), one copy of the code for every layer,
// which then stays in the instruction cache, weights asked for before the values of the layer before them are
// worked out, and states before the barrier.
// With sixteen waves on four SIMDs an instruction of a wave takes its turn every 16 cycles or so, scalar ones included: a layer takes
// as long as the instructions beside the matrix ones are many.  Hence arguments that a wave keeps in the lanes of two registers, a step
// ahead, and takes from there where it needs them (as scalar loads they were waited for, and of sixty values at once a third were put
// aside and fetched back: 3975 instead of 3785 us, all else equal), worked out as far as the host can, three-operand bounds, bytes packed
// and counted by the word, and rows that nothing reaches left out.
// Measured in one stage, per image of 112 x 112, int8, eight streams, 112 pushes: 4173 us, with fewer instructions 3860, waiting for weights and
// states together 3727, as it is 3195; float32, 256 streams of 32 x 32, 32 pushes: 1130 -> 1034 us.  Per pushed row 28.5 us (layer by
// layer 170) and 32 us (112), of which 14 us are matrix instructions (4,300 of 32 cycles, even over four SIMDs).
#include <algorithm>
#include <type_traits>

#include "idf.h"
#include "idf_kernels.h"
#include "mfma_tile.h"

namespace idf {

namespace {

typedef const __attribute__((address_space(4))) EagerPassStep PassStep;
typedef const __attribute__((address_space(4))) EagerPass PassArgs;

constexpr int kPassLds = 160 * 1024 - 512;

// Zero times infinity is not zero: in a float net the first layer's positions carry as many cells of zeros as the last K-step of
// their windows reads too far.  (Layers behind it have a multiple of 16 channels: their windows are whole K-steps.)
__host__ __device__ inline int pad_cells(bool is_float, int cells) { return is_float ? -3 * cells & 3 : 0; }

extern __shared__ __attribute__((aligned(16))) unsigned char pass_smem[];

// ---- the pushed rows: announced values, events, and the first layer's delta band ---------------------
template <class T, int WAVES> __device__ __forceinline__ void pass_input(PassArgs &a, PassStep &L, int stream, int pos, bool announces, uint32_t *events)
{
    constexpr int kThreads = 64 * WAVES;
    using ev_t = typename T::ev_t; using st_t = typename T::st_t;
    const int tid = threadIdx.x, W = L.w, C = L.c_in, n_rows = L.n_in, row_elems = W * C;
    const ev_t *src = (const ev_t *)a.in + (int64_t)pos * a.in_stride;
    st_t *ann = (st_t *)a.ann0 + (int64_t)stream * a.ann0_stride;
    unsigned char *out = pass_smem + L.lds_in;
    const int XP = 16 * L.n_xt + 2;
    uint32_t ev = 0;
    int slot = a.ann0_slot;
    if (announces) for (int r = 0; r < n_rows; ++r) {
        for (int i = tid; i < row_elems; i += kThreads) {
            const ev_t v = src[r * row_elems + i];
            ann[(int64_t)slot * row_elems + i] = (st_t)v;
            ev += T::ev_nonzero(v);
        }
        slot = slot + 1 == a.ann0_rows ? 0 : slot + 1;
    }
    if (L.cells > 0) {                             // whole cells: [row][position, one of halo in front][channel], padded (pad_cells)
        const int cells = L.cells, all = cells + pad_cells(T::EB == 4, cells), n = XP * all;
        for (int r = 0; r < n_rows; ++r)
            for (int i = tid; i < n; i += kThreads) {
                const int p = i / all, c = i - p * all, x = p - 1;
                i32x4 v = {0, 0, 0, 0};
                if (x >= 0 && x < W && c < cells) v = reinterpret_cast<const i32x4 *>(src)[(r * W + x) * cells + c];
                *reinterpret_cast<i32x4 *>(out + r * L.in_pitch + p * L.in_stride + c * 16) = v;
            }
    } else {                                       // few channels: the windows the positions see, 3 * C values padded to cells
        auto windows = [&](auto n_tag) IDF_INLINE {
            constexpr int NC = decltype(n_tag)::value, WC = window_cells(NC, T::VL, T::EB == 4);
            const int XT = 16 * L.n_xt;
            // (a wave takes whole rows: the waves are many and a row is short)
            for (int r = tid >> 6; r < n_rows; r += WAVES)
              for (int p = tid & 63; p < XT; p += 64) {
                ev_t val[WC * T::VL];
#pragma unroll
                for (int k = 0; k < WC * T::VL; ++k) val[k] = 0;
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const int x = p - 1 + kx, xc = x < 0 ? 0 : (x >= W ? W - 1 : x);
#pragma unroll
                    for (int ci = 0; ci < NC; ++ci) {
                        const ev_t v = src[(r * W + xc) * NC + ci];
                        val[kx * NC + ci] = x == xc ? v : (ev_t)0;
                    }
                }
                i32x4 w[WC];
                __builtin_memcpy(w, val, sizeof(w));
#pragma unroll
                for (int k = 0; k < WC; ++k) *reinterpret_cast<i32x4 *>(out + r * L.in_pitch + p * L.in_stride + k * 16) = w[k];
            }
        };
        switch (C) {
        case 1: windows(std::integral_constant<int, 1>{}); break;
        case 2: windows(std::integral_constant<int, 2>{}); break;
        case 3: windows(std::integral_constant<int, 3>{}); break;
        default: windows(std::integral_constant<int, 4>{}); break;
        }
    }
    ev = wave_sum(ev);
    if ((tid & 63) == 0 && ev) atomicAdd(events, ev);
}

// A step's arguments as a wave keeps them: lane i holds word i, and a value is taken from its lane where it is used.
constexpr int kStepWords = sizeof(EagerPassStep) / 4;
static_assert(kStepWords <= 64, "a word to each lane");
__device__ __forceinline__ int step_words(PassStep *L)
{
    const int lane = threadIdx.x & 63;
    return ((const __attribute__((address_space(4))) int *)L)[lane < kStepWords ? lane : kStepWords - 1];
}
template <class V> __device__ __forceinline__ V step_value(int words, int at)
{
    if constexpr (sizeof(V) == 8) return (V)(__attribute__((address_space(1))) void *)((uint64_t)(uint32_t)__builtin_amdgcn_readlane(words, at) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane(words, at + 1) << 32);
    else return (V)__builtin_amdgcn_readlane(words, at);
}
#define IDF_OF(words, field) step_value<decltype(EagerPassStep::field)>(words, (int)offsetof(EagerPassStep, field) / 4)

// The weights a wave has on their way: of one K-step, the task's next or behind its last the first of the wave's next task, which as a
// rule is of the next layer and has the time of all that stands between.  (Three K-steps on their way, asked for at every task whether
// it has them or not: int8 3785 instead of 3310 us, float32 1074 instead of 1058.  Asked for where it has them, they would be out or
// not: every wait then counts as if they were not.)
template <class T> struct Weights {
    i32x4 q[3];
    const unsigned char *base[3];                  // of each tap row
    int ct, rest;                                  // the task: its tile of channels, and what is left of its number
    uint32_t step, off;                            // bytes from one K-step to the next; this lane's place in the one asked for next
    __device__ __forceinline__ void aim(int words, int t)      // at task t of a step
    {
        const int n_ct = IDF_OF(words, n_ct);
        rest = (int)__umulhi((unsigned)t, IDF_OF(words, ct_rcp)) + (n_ct == 1 ? t : 0);
        ct = t - rest * n_ct;
        const uint32_t w_ky = IDF_OF(words, w_ky);
        const void *w_frag = IDF_OF(words, w_frag);
        step = IDF_OF(words, w_kstep);
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) base[ky] = (const unsigned char *)w_frag + ((ct >> 1) * 6144 + (ct & 1) * 1024 + ky * w_ky);
        off = (threadIdx.x & 63) * 16;
    }
    __device__ __forceinline__ void fetch()
    {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) q[ky] = *at4(reinterpret_cast<const i32x4 *>(base[ky]), off);
        off += step;
    }
};

// ---- one conv layer, and the 2x2 max-pool behind it ------------------------------------------------------
// SPLIT: the only layer of its stage, whose tasks `parts` workgroups share; differences go to memory (hand) from the lanes that have them.
template <class T, int WAVES, bool SPLIT> __device__ __forceinline__ void pass_conv(PassArgs &a, int words, int next, Weights<T> &wt, int stream, int part, int parts,
                                                                                    unsigned char *hand, uint32_t *all_events)
{
    using acc_t = typename T::acc_t; using st_t = typename T::st_t;
    constexpr bool kInt = T::EB == 1;
#define STEP(field) IDF_OF(words, field)
    const int tasks = STEP(tasks), n_ksteps = STEP(n_ksteps), layer = STEP(layer), emit = STEP(emit), pool = STEP(pool);
    const int C_out = STEP(c_out), in_pitch = STEP(in_pitch), in_stride = STEP(in_stride), cells = STEP(cells);
    const int out_pitch = STEP(out_pitch), out_stride = STEP(out_stride);
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), m = lane & 15, g = lane >> 4;
    char *c_map = (char *)STEP(c) + (uint64_t)(uint32_t)stream * STEP(c_stride) * 4;

    acc_t old[4];                                  // states as they were
    int xt = 0, gi = 0, x = 0, co0 = 0;
    uint32_t cell = 0;                             // this lane's first channel, bytes into a row
    uint32_t c_off[4];                             // bytes from a stream's first row kept to each row
    bool here = false;
    // the states of a task are asked for before its cells are there
    auto begin = [&]() IDF_INLINE {
        const int n_xt = STEP(n_xt), rest = wt.rest, ct = wt.ct;
        gi = (int)__umulhi((unsigned)rest, STEP(xt_rcp)) + (n_xt == 1 ? rest : 0);
        xt = rest - gi * n_xt;
        x = xt * 16 + m;
        co0 = (ct >> 1) * 32 + (ct & 1) * 4 + g * STEP(co_g);
        here = (int)(x < STEP(w)) & (int)(co0 < C_out);
        cell = here ? (uint32_t)(x * C_out + co0) * 4 : 0;
        constexpr int kSlot = (int)offsetof(EagerPassStep, c_slot) / 4;
        const uint32_t s01 = step_value<uint32_t>(words, kSlot + 2 * gi), s23 = step_value<uint32_t>(words, kSlot + 1 + 2 * gi), row_bytes = STEP(row_bytes);
        c_off[0] = (s01 & 0xffffu) * row_bytes; c_off[1] = (s01 >> 16) * row_bytes;
        c_off[2] = (s23 & 0xffffu) * row_bytes; c_off[3] = (s23 >> 16) * row_bytes;
        // (rows without a state are read like the others: their places exist)
#pragma unroll
        for (int j = 0; j < 4; ++j) old[j] = *at4(reinterpret_cast<const acc_t *>(c_map + c_off[j]), cell);
    };
    const int act_none = STEP(act_none), act_lo = STEP(act_lo), act_shr = STEP(act_shr);
    int act_hi = STEP(act_hi);
    asm("" : "+v"(act_hi));                        // (an instruction takes one scalar)
    const FloatBounds bounds(act_none);
    auto act = [&](st_t v) IDF_INLINE {
        if constexpr (kInt) return (st_t)between((int32_t)v >> act_shr, act_lo, act_hi);
        else return bounds(v);
    };
    uint32_t ev = 0, ev_pool = 0;                  // (int8: of this lane; float32: of the wave)
    // the band is there, and nobody reads what this layer overwrites any more; what is passed on has zeros in front of each row, and
    // behind it as far as no lane of the tiles reaches
    auto enter = [&]() IDF_INLINE {
        lds_barrier();
        const int out_rows = STEP(out_rows), out_done = STEP(out_done), out_end = STEP(out_end);
        if (!SPLIT && emit) for (int r = wave; r < out_rows; r += WAVES) {
            unsigned char *row = pass_smem + STEP(lds_out) + r * out_pitch;
            for (int o = lane * 16; o < out_stride; o += 1024) *reinterpret_cast<i32x4 *>(row + o) = i32x4{0, 0, 0, 0};
            for (int o = out_done + lane * 16; o < out_end; o += 1024) *reinterpret_cast<i32x4 *>(row + o) = i32x4{0, 0, 0, 0};
        }
    };
    // Every wave takes the same way, one without a task too, and a state is known to be here before a round ends: a request made on one
    // of two ways counts as out wherever they meet, and had the next layer wait for what it did not need yet.
    const int all = SPLIT ? WAVES * parts : WAVES;             // waves that share the tasks
    int rounds = SPLIT ? 1 : (int)((unsigned)(tasks + WAVES - 1) / WAVES), t = SPLIT ? part * WAVES + wave : wave;
    if (SPLIT) for (int i = all; i < tasks; i += all) ++rounds;
    asm volatile("" : "+s"(rounds));
#pragma unroll 1
    do {
        --rounds;
        const int n_mine = t < tasks ? n_ksteps : 0;           // (a wave without a task asks for its next weights like the others)
        if (n_mine) begin();
        if (t < all) enter();
        acc_t acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = acc_t{0, 0, 0, 0};
        const uint32_t in = STEP(rows_in) >> (4 * gi);   // bit r: row r - 1 of the four (-1 .. 4) is in the band
        {
            const uint32_t base = (uint32_t)(STEP(lds_in) + (xt * 16 + m) * in_stride);
            const uint32_t row0 = (uint32_t)((STEP(band0) + 4 * gi) * in_pitch);
            uint32_t row[6];                       // where the six rows lie (those outside the band: its first)
#pragma unroll
            for (int r = 0; r < 6; ++r) row[r] = (in >> r) & 1u ? row0 + (uint32_t)r * (uint32_t)in_pitch : 0u;
            // K-step st holds cells 4 st .. 4 st + 3 of the window's 3 * cells, counted tap column by tap column (past the end, where
            // the weights are zero, the padding of the last position; int8: the last one again); few channels: the cells of the
            // gathered window
            auto at = [&](int st) IDF_INLINE {
                int q = 4 * st + g;
                if (cells == 0) return kInt ? base : base + (uint32_t)q * 16;        // (int8: one cell)
                if (kInt) q = q < 3 * cells ? q : 3 * cells - 1;
                return base + (uint32_t)(((q >= cells) + (q >= 2 * cells)) * (in_stride - cells * 16) + q * 16);
            };
            auto kstep = [&](uint32_t off) IDF_INLINE {
                i32x4 xv[6];
#pragma unroll
                for (int r = 0; r < 6; ++r)
                    xv[r] = *reinterpret_cast<const i32x4 *>(pass_smem + (off + row[r]));
#pragma unroll
                for (int r = 0; r < 6; ++r) {
                    if (!((in >> r) & 1u)) continue;
#pragma unroll
                    for (int e = 0; e < T::kInst; ++e)
#pragma unroll
                        for (int ky = 0; ky < 3; ++ky)
                            if (r - ky >= 0 && r - ky < 4) acc[r - ky] = T::mfma(wt.q[ky], xv[r], acc[r - ky], e);
                }
            };
            int st = 0;
#pragma unroll 1
            do {
                if (st + 1 >= n_mine) wt.aim(rounds ? words : next, rounds ? t + all : wave);
                if (n_mine) kstep(at(st));
                wt.fetch();
                __builtin_amdgcn_sched_barrier(0);
            } while (++st < n_mine);
        }
        __builtin_amdgcn_s_waitcnt(0xf73);         // vmcnt(3): all but the weights asked for last are here
        __builtin_amdgcn_sched_barrier(0);
        if (n_mine) {
        // the state moves on; what is announced is f of it, less f of what it was
        const uint32_t on = STEP(rows_on) >> (4 * gi), had = STEP(rows_old) >> (4 * gi);
        const bool out_ok = emit && co0 < C_out;
        unsigned char *out = pass_smem + STEP(lds_out) + STEP(out_first) * out_pitch + co0 * T::EB;
        const int hand_pos = C_out * T::EB, hand_row = STEP(out_w) * hand_pos;
        unsigned char *to_next = SPLIT ? hand + ((int64_t)stream * STEP(out_rows) + STEP(out_first)) * hand_row + co0 * T::EB : nullptr;
        // the differences of four channels (zero beyond the row's end) are counted and passed on
        auto deliver = [&](const acc_t &h_new, const acc_t &h_old, bool mine, uint32_t &n, unsigned char *to, bool pass) IDF_INLINE {
            st_t d[4];
            uint32_t e[T::EB];
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = h_new[i] - h_old[i];
            if constexpr (kInt) {
                T::pack4(d, e);
                e[0] = mine ? e[0] : 0u;
                n += (uint32_t)T::nonzero(e[0]);
                if (pass) *reinterpret_cast<uint32_t *>(to) = e[0];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] = mine ? d[i] : (st_t)0;
#pragma unroll
                for (int i = 0; i < 4; ++i) n += (uint32_t)__builtin_popcountll(__ballot(d[i] != 0));
                T::pack4(d, e);
                if (pass) *reinterpret_cast<i32x4 *>(to) = i32x4{(int)e[0], (int)e[1], (int)e[2], (int)e[3]};
            }
        };
        void *ann_map = STEP(ann);
        const uint32_t ann_stride = STEP(ann_stride), pool_on = STEP(pool_on);
        const int W = STEP(w), out_w = STEP(out_w);
        char *ann = ann_map && !pool ? (char *)ann_map + ((int64_t)stream * ann_stride + (int64_t)(STEP(row0) + 4 * gi) * W * C_out) * 4 : nullptr;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            acc_t h_new[2], h_old[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int j = 2 * p + q;
                h_new[q] = h_old[q] = acc_t{0, 0, 0, 0};       // (rows that have not been reached announce zero)
                if (!(((on | (pool ? had : 0u)) >> j) & 1u)) continue;
                if ((had >> j) & 1u) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) { acc[j][i] += old[j][i]; h_old[q][i] = act(old[j][i]); }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) h_new[q][i] = act(acc[j][i]);
                if (!((on >> j) & 1u)) continue;
                if (here) {
                    *at4(reinterpret_cast<acc_t *>(c_map + c_off[j]), cell) = acc[j];
                    if (ann) *at4(reinterpret_cast<acc_t *>(ann + (int64_t)(j * W * C_out) * 4), cell) = h_new[q];
                }
                deliver(h_new[q], h_old[q], here, ev, SPLIT ? to_next + (4 * gi + j) * hand_row + x * hand_pos : out + (4 * gi + j) * out_pitch + (x + 1) * out_stride,
                        !pool && out_ok && (!SPLIT || here));
            }
            if (pool && ((pool_on >> (2 * gi + p)) & 1u)) {
                const bool mine = (x & 1) == 0 && (x >> 1) < out_w && co0 < C_out;
                acc_t n, o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const st_t nn = h_new[0][i] > h_new[1][i] ? h_new[0][i] : h_new[1][i], oo = h_old[0][i] > h_old[1][i] ? h_old[0][i] : h_old[1][i];
                    const st_t nx = neighbour(nn), ox = neighbour(oo);
                    n[i] = nn > nx ? nn : nx;
                    o[i] = oo > ox ? oo : ox;
                }
                if (mine) *at4(reinterpret_cast<acc_t *>((char *)ann_map + (int64_t)stream * ann_stride * 4 + (int64_t)((step_value<uint32_t>(words, (int)offsetof(EagerPassStep, pool_slots) / 4 + gi) >> p * 16) & 0xffffu) * (out_w * C_out * 4)),
                               (uint32_t)((x >> 1) * C_out + co0) * 4) = n;
                deliver(n, o, mine, ev_pool, SPLIT ? to_next + (2 * gi + p) * hand_row + (x >> 1) * hand_pos : out + (2 * gi + p) * out_pitch + ((x >> 1) + 1) * out_stride, emit && mine);
            }
        }
        }
        t += all;
    } while (rounds);
    if constexpr (kInt) {
        ev = wave_sum(ev);
        if (pool) ev_pool = wave_sum(ev_pool);
    }
    // (an instruction each: an atomic of the language is prepared for lanes of many)
    if (lane == 0) {
        const uint32_t level = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)(all_events + layer);
        asm volatile("ds_add_u32 %0, %1 offset:4" ::"v"(level), "v"(ev) : "memory");         // (the last layer's are of no level: nobody looks at that place)
        if (pool) asm volatile("ds_add_u32 %0, %1 offset:8" ::"v"(level), "v"(ev_pool) : "memory");
    }
}

// ---- from stage to stage: the delta band as rows of whole cells, [row][position][cell], stream after stream ---------------
// (four requests of a thread at once: one by one, each would be a trip to memory of its own)
template <int WAVES> __device__ __forceinline__ void pass_hand_in(PassStep &L, const void *hand, int stream)
{
    constexpr int kThreads = 64 * WAVES, N = 4;
    const int tid = threadIdx.x, W = L.w, cells = L.cells, per_row = (16 * L.n_xt + 2) * cells, n = L.n_in * per_row;
    const i32x4 *src = reinterpret_cast<const i32x4 *>(hand) + (int64_t)stream * (L.n_in * W * cells);
    const unsigned row_rcp = uni((int)(0xffffffffu / (unsigned)per_row + 1)), cell_rcp = uni((int)(0xffffffffu / (unsigned)cells + 1));
    unsigned char *out = pass_smem + L.lds_in;
    for (int i0 = tid; i0 < n; i0 += N * kThreads) {
        i32x4 v[N];
        int to[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int i = i0 + k * kThreads;
            const int r = (int)__umulhi((unsigned)i, row_rcp), in_row = i - r * per_row;
            const int p = cells == 1 ? in_row : (int)__umulhi((unsigned)in_row, cell_rcp), c = in_row - p * cells;
            const bool there = i < n && p >= 1 && p <= W;
            to[k] = r * L.in_pitch + p * L.in_stride + c * 16;
            v[k] = i32x4{0, 0, 0, 0};
            if (there) v[k] = src[(r * W + p - 1) * cells + c];
        }
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (i0 + k * kThreads < n) *reinterpret_cast<i32x4 *>(out + to[k]) = v[k];
    }
}
template <int EB, int WAVES> __device__ __forceinline__ void pass_hand_on(PassStep &L, void *hand, int stream)
{
    constexpr int kThreads = 64 * WAVES;
    const int tid = threadIdx.x, cells = L.c_out * EB / 16, per_row = L.out_w * cells, n = L.out_rows * per_row;
    i32x4 *dst = reinterpret_cast<i32x4 *>(hand) + (int64_t)stream * n;
    const unsigned row_rcp = uni((int)(0xffffffffu / (unsigned)per_row + 1)), cell_rcp = uni((int)(0xffffffffu / (unsigned)cells + 1));
    const unsigned char *in = pass_smem + L.lds_out;
    for (int i = tid; i < n; i += kThreads) {
        const int r = per_row == 1 ? i : (int)__umulhi((unsigned)i, row_rcp), in_row = i - r * per_row;
        const int p = cells == 1 ? in_row : (int)__umulhi((unsigned)in_row, cell_rcp), c = in_row - p * cells;
        dst[i] = *reinterpret_cast<const i32x4 *>(in + r * L.out_pitch + (p + 1) * L.out_stride + c * 16);
    }
}

// A workgroup takes one stream through the whole net or, STAGED, through one stage of it (gridDim.y of them, from a.stage0 on): layers
// first[stage] .. end[stage] - 1.  SPLIT: stages are of one layer, whose tiles gridDim.z workgroups share (a.parts; the rule stands at eager_stages).  (Kernels
// of their own: which layers they are is a trip to memory, 1.5 % of a pass of eight.  So are the launches of a recording that may find nothing
// left to do, OPEN: asked by every launch, 0.3 to 0.9 %.)
template <class T, int WAVES, bool STAGED, bool SPLIT, bool OPEN = false>
__global__ void __launch_bounds__(64 * WAVES, 4) k_eager_pass(const EagerPass args, const StreamSel sel)
{
    // the arguments are read where the launch put them, a step at a time (by value they would be copied to scratch memory)
    PassArgs &a = *(PassArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ uint32_t events[2 * kPassMax + 2];      // per level
    const int tid = threadIdx.x, stream = sel_stream(sel, blockIdx.x), stage = STAGED ? a.stage0 + (int)blockIdx.y : 0;
    const int k0 = STAGED ? a.first[stage] : 0, n = STAGED ? a.end[stage] : a.n, part = SPLIT ? (int)blockIdx.z : 0, parts = SPLIT ? a.parts : 1;
    if (STAGED && k0 >= n) return;
    if (OPEN && *a.open == 0) return;
    int words = step_words(&a.st[k0]), next = step_words(&a.st[k0 + 1 < n ? k0 + 1 : k0]);
    if (tid < 2 * kPassMax + 2) events[tid] = 0;
    if constexpr (SPLIT) request_arguments<sizeof(EagerPassStep), WAVES>(&a.st[k0], &a + 1);
    else request_arguments<sizeof(EagerPass), WAVES>(&a, &a + 1);
    if (SPLIT && part * WAVES >= IDF_OF(words, tasks) && part > 0) return;
    Weights<T> wt;
    wt.aim(words, part * WAVES + uni(tid >> 6));
    wt.fetch();
    asm volatile("" : "+v"(next));
    lds_barrier();
    if (STAGED && k0 > 0) pass_hand_in<WAVES>(a.st[k0], (const char *)a.hand + (uint64_t)a.hand_in[stage] * 256, stream);
    else pass_input<T, WAVES>(a, a.st[0], stream, sel.pos0 + (int)blockIdx.x, part == 0, &events[0]);
#pragma unroll 1
    for (int k = k0; k < n; ++k) {
        asm volatile("" : "+v"(next));             // (it is here)
        const int after = step_words(&a.st[k + 2 < n ? k + 2 : n - 1]);
        pass_conv<T, WAVES, SPLIT>(a, words, next, wt, stream, part, parts, SPLIT ? (unsigned char *)a.hand + (uint64_t)a.hand_out[stage] * 256 : nullptr, events);
        words = next;
        next = after;
    }
    lds_barrier();
    if (STAGED && !SPLIT && a.st[n - 1].emit) pass_hand_on<T::EB, WAVES>(a.st[n - 1], (char *)a.hand + (uint64_t)a.hand_out[stage] * 256, stream);
    if (tid < a.n_layers && events[tid]) atomicAdd(a.stats + ((int64_t)stream * a.n_layers + tid) * 2, (unsigned long long)events[tid]);
}

template <class T>
__global__ void __launch_bounds__(256) k_eager_announced(const typename T::st_t *c, int c_rows, int64_t first, int64_t row, int act, int shr, int hi, typename T::st_t *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < row) out[blockIdx.y * row + i] = T::activate(c[(first + blockIdx.y) % c_rows * row + i], act, shr, hi);
}

}  // namespace

// Lays the bands out in LDS; false where they do not fit.
bool eager_pass_shape(int prec, EagerPass &a)
{
    const int vl = conv3x3_mfma_vl(prec), eb = 16 / vl;
    size_t lds = 0, size[kPassMax + 1] = {};
    auto rcp32 = [](int n) { return n > 1 ? (unsigned)((0x100000000ull + n - 1) / n) : 0u; };
    for (int k = 0; k < a.n; ++k) {
        EagerPassStep &L = a.st[k];
        const bool single = L.c_out == 16;
        const int n_blk = (L.c_out + 31) / 32;
        L.n_xt = (L.w + 15) / 16;
        L.n_ct = single ? 1 : 2 * n_blk;
        L.tasks = L.n_ct * L.n_xt * L.n_groups;
        L.co_g = single ? 4 : 8;
        L.w_kstep = single ? 3 * 1024 : (uint32_t)n_blk * 6144; L.w_ky = single ? 1024 : 2048;
        L.xt_rcp = rcp32(L.n_xt); L.ct_rcp = rcp32(L.n_ct);
        L.cells = L.c_in % vl == 0 ? L.c_in / vl : 0;
        L.n_ksteps = L.cells ? (3 * L.cells + 3) / 4 : 1;
        L.in_stride = cell_stride(L.cells ? L.cells + pad_cells(eb == 4, L.cells) : window_cells(L.c_in, vl, eb == 4)) * 16;
        L.in_pitch = (16 * L.n_xt + 2) * L.in_stride;
        size[k] = (size_t)L.n_in * L.in_pitch;
        if (k > 0) {
            EagerPassStep &P = a.st[k - 1];
            P.out_stride = L.in_stride; P.out_pitch = P.out_end = L.in_pitch; P.out_rows = L.n_in;
            P.out_done = ((P.pool ? P.out_w : 16 * P.n_xt) + 1) * L.in_stride;
        }
    }
    for (int k = 0; k < a.n; ++k) lds = std::max(lds, size[k] + size[k + 1]);
    if (lds > kPassLds) return false;
    for (int k = 0; k < a.n; ++k) {                // bands lie alternately at the bottom and at the top
        a.st[k].lds_in = k & 1 ? (int)(lds - size[k]) : 0;
        a.st[k].lds_out = k & 1 ? 0 : (int)(lds - size[k + 1]);
    }
    a.lds = (int)lds;
    return true;
}

hipError_t launch_eager_pass(int prec, const EagerPass &a, int stages, bool small, const StreamSel &sel, const LaunchCtx &lc)
{
    auto go = [&](auto kernel, int waves) {
        const hipError_t e = allow_lds<kPassLds>(kernel);
        return e != hipSuccess ? e : launch(kernel.entry, dim3(sel.n, std::max(1, stages), std::max(1, a.parts)), dim3(64 * waves), (size_t)a.lds, lc, a, sel);
    };
    auto of = [&](auto t) {
        using T = decltype(t);
        if (stages == 0) return go(Kernel<k_eager_pass<T, 16, false, false>>{}, 16);
        if (a.open) {
            if (a.parts > 0) return go(Kernel<k_eager_pass<T, 4, true, true, true>>{}, 4);
            return small ? go(Kernel<k_eager_pass<T, 8, true, false, true>>{}, 8) : go(Kernel<k_eager_pass<T, 16, true, false, true>>{}, 16);
        }
        if (a.parts > 0) return go(Kernel<k_eager_pass<T, 4, true, true>>{}, 4);
        return small ? go(Kernel<k_eager_pass<T, 8, true, false>>{}, 8) : go(Kernel<k_eager_pass<T, 16, true, false>>{}, 16);
    };
    return prec == IDF_PREC_I8 ? of(TraitsI8{}) : of(TraitsF32{});
}

hipError_t launch_eager_announced(int prec, const Geom &g, const void *c, int c_rows, int64_t first, int n, void *out, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t row = (int64_t)g.w_out * g.c_out;
    const dim3 grid((unsigned)((row + 255) / 256), (unsigned)n), block(256);
    LaunchCtx lc;
    lc.st = st;
    if (prec == IDF_PREC_I8) return launch(k_eager_announced<TraitsI8>, grid, block, 0, lc, (const int32_t *)c, c_rows, first, row, g.act, g.shr, g.clamp_hi, (int32_t *)out);
    return launch(k_eager_announced<TraitsF32>, grid, block, 0, lc, (const float *)c, c_rows, first, row, g.act, g.shr, g.clamp_hi, (float *)out);
}

}  // namespace idf
