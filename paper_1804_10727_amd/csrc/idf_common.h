// Shared between the host side of the library and its kernels: layer geometry, the
// data-independent row schedule, and the argument blocks handed to the kernels.
#pragma once

#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define IDF_HD __host__ __device__ inline
#else
#define IDF_HD inline
#endif

namespace idf {

constexpr int kMaxLayers = 32;
constexpr int kSelIds = 16;    // stream ids carried by value in one launch (kept small: kernel arguments are fetched from memory)

struct Geom {
    int kind;            // IDF_CONV / IDF_MAXPOOL
    int c_in, c_out, k_h, k_w, s_h, s_w, p_h, p_w;
    int act, shr, clamp_hi;
    int h_in, w_in;      // h_in = 0: unbounded
    int h_out, w_out;    // h_out = 0: unbounded
};

IDF_HD int out_size(int n, int k, int s, int p)
{
    int t = n + 2 * p - k;
    return t < 0 ? 0 : t / s + 1;
}

// Number of output rows of a layer that are final once it has received rows 0..y-1 of its
// input.  Output row o needs input rows o*s-p .. o*s-p+k-1 (clipped to the sample), so it is
// final when y >= o*s-p+k, and every row is final once the whole sample (h_in rows) is in:
// the bottom padding contributes nothing.
IDF_HD int64_t rows_final(const Geom &g, int64_t y)
{
    if (g.h_in > 0 && y >= g.h_in) return g.h_out;
    int64_t t = y + g.p_h - g.k_h;
    int64_t n = t < 0 ? 0 : t / g.s_h + 1;
    if (g.h_out > 0 && n > g.h_out) n = g.h_out;
    return n;
}

// One past the last output row that input rows 0..y-1 have contributed to (first input row
// of output row o is o*s-p).
IDF_HD int64_t rows_touched(const Geom &g, int64_t y)
{
    if (y <= 0) return 0;
    int64_t n = (y - 1 + g.p_h) / g.s_h + 1;
    if (g.h_out > 0 && n > g.h_out) n = g.h_out;
    return n;
}

// Stream selection of one launch: either the contiguous ids base .. base+n-1 or n ids by value.
struct StreamSel {
    int n;
    int base;            // >= 0: contiguous; -1: use ids[]
    int pos0;            // position of the first selected stream in the caller's id list
    int ids[kSelIds];
};

__host__ __device__ inline int sel_stream(const StreamSel &s, int i) { return s.base >= 0 ? s.base + i : s.ids[i]; }

// One step of one conv layer for a group of streams that are all at the same row:
// input rows [y0, y0+cnt) arrive; output rows [o_lo, o_hi) are touched; of those
// [o_lo, o_fin) become final and are emitted, the rest go back to the ring.
struct ConvStep {
    Geom g;
    int layer;
    int64_t y0;
    int cnt;
    int64_t o_lo, o_fin, o_hi;
    int ring_rows;               // slots of the ring (k_h)
    // input rows: [stream or position][row - in_row0][w_in][c_in]
    const void *in;
    int64_t in_stream_stride;    // elements
    int64_t in_row0;             // input row held in slot 0
    int in_by_position;          // 1: index by position in the caller's list (network input)
    // state ring [stream][slot][w_out][c_out], slot = o mod ring_rows
    void *ring;
    int64_t ring_stream_stride;
    // destination of emitted rows: next layer's transit rows (slot = o - dst_row0) or, for the
    // last layer, the output area (slot = (dst_slot0 + o - dst_row0) mod out_cap)
    void *dst;
    int64_t dst_stream_stride;
    int64_t dst_row0, dst_slot0;
    int dst_ring;                // > 0: the next layer keeps its input rows in a ring of that many slots, slot = (dst_slot0 + o - dst_row0) mod dst_ring
    int to_output;
    int64_t out_cap;
    const void *w;               // [k_h][k_w][c_in][c_out]
    const void *bias;            // [c_out] or null
    unsigned long long *stats;   // [stream][layer][2]: events_in, macs
    int n_layers;
    int tile_x, tile_c, cells_per_thread;
    // A pixel segment of the network input (one row, cnt == 1): only columns [x_lo, x_hi) of the row are there,
    // column x_lo first in the buffer; x_hi == 0: the whole row.  cont: an earlier segment of the same row has
    // started the rows it touches, so every cell continues from the ring.
    int x_lo, x_hi, cont;
};

struct PoolStep {
    Geom g;
    int layer;
    int64_t y0;
    int cnt;
    int64_t o_lo, o_fin;         // output rows emitted: [o_lo, o_fin)
    int hold_new;                // 1: the last new row is the even row of a pair: hold it
    const void *in;
    int64_t in_stream_stride;
    int64_t in_row0;
    int in_by_position;
    void *held;                  // [stream][w_in][c]
    int64_t held_stream_stride;
    void *dst;
    int64_t dst_stream_stride;
    int64_t dst_row0, dst_slot0;
    int dst_ring;                // as in ConvStep
    int to_output;
    int64_t out_cap;
    unsigned long long *stats;
    int n_layers;
};

// Output rows of one conv layer on the matrix cores (k_conv3x3_mfma.hip).  A layer keeps the rows of its
// input that some output row still needs, as events, in a ring; an output row of c is formed in
// registers once its last input row has arrived, activated and emitted.
constexpr int kRowLaunchRows = 16;     // arriving rows one launch takes at most (longer pushes are several launches)

enum { kRowTake = 0,                   // no convolution: rows of the caller go into the ring and are counted
       kRowSmall1, kRowSmall2,         // a wave does 16 positions x 16 channels of 1 / 2 output rows
       kRowWide2 };                    // a wave does 32 positions x 32 channels of 2 output rows

struct RowStep {
    int form;                          // kRow*
    int tiles;                         // workgroups per stream
    int w, h;                          // positions per row, rows per sample (input and output alike)
    int c_in, c_out;
    int cells;                         // 16-byte cells per position (0: one to four channels)
    int y0, n_rows;                    // first output row (index in the sample) and how many; kRowTake: input rows
    int slot0;                         // ring slot of input row y0 - 1 (kRowTake: of row y0), whether that row exists or not
    int ring_rows;                     // slots of the ring
    int y_new;                         // input rows from this one on are in the caller's buffer, the others in the ring
    int y_save;                        // kRowTake: rows from this one on go into the ring
    int x_lo, x_hi;                    // kRowTake: columns of the row that are given (a pixel segment)
    int wc_log;                        // log2 of the waves of a workgroup that lie side by side along the channels
    int n_xt, n_cg;                    // position tiles of a row, channel groups
    unsigned xt_rcp, cg_rcp;           // ceil(2^32 / n) of those (0 for one)
    int nb, row_pos;                   // blocks of 64 cells per row of a stretch; positions those cover: what a row takes in LDS
    unsigned cells_rcp;                // ceil(65536 / cells)
    int stride, row_pitch;             // bytes in LDS from one position, and one row of a stretch, to the next
    int n_ct, co_g;                    // tiles of 16 output channels; channels from one group of lanes to the next
    int n_ksteps;                      // K-steps of the contraction
    unsigned w_kstep, w_ky;            // bytes from one K-step, and one tap row, to the next in the packed weights
    int act, shr, clamp_hi;
    int pool;                          // 1: 2x2 max-pool behind the layer
    int pool_from;                     // output rows before this one have been counted as the pool's events already
    int pool_emit;                     // 0: only count the pool's events, emit nothing
    int to_output;
    int dst_slot0, dst_rows;           // slot of the first emitted row, slots of the destination
    int layer, pool_layer, next_layer, next_c_out, n_layers;     // next_layer: the layer whose events the emitted rows are (-1: it counts them itself)
    int ev_limit;                      // a row's stretch of 32 positions with at most this many events goes the event path (0: never; at most half the list's length)
    int64_t in_stride, new_stride;     // elements per stream of the ring / of the caller's buffer
    const void *in_ring, *in_new;
    void *dst;
    int64_t dst_stride;
    const void *wfrag;                 // fragment-ordered weights
    const void *w_ev;                  // int8 nets: weights for the event path, [kx][c_in][c_out_pad] words of the three ky taps
    const void *bias;
    unsigned long long *stats;
    unsigned long long *issued;        // [stream][layer] multiply-adds issued by the matrix instructions, or null
};

// Steps of several layers for one launch of the matrix-core kernel.
constexpr int kRowUnits = 8;           // conv layers one launch can hold
constexpr int kRowBatchMax = kRowUnits + 1;
struct RowBatch {
    int n;
    RowStep st[kRowBatchMax];
};
static_assert(sizeof(RowBatch) + sizeof(StreamSel) <= 4096, "a launch's arguments must fit the kernel-argument segment");

struct CopyOut {
    const void *src;             // output area [stream][out_cap][row_elems]
    int64_t src_stream_stride;
    int64_t out_cap;
    void *dst;                   // [position][max_rows][row_elems]
    int64_t dst_stream_stride;
    int64_t row_elems;
    int elem_bytes;
};

// One layer's step in eager emission: output rows [o_lo, o_hi) take in the delta rows
// [i_lo, i_hi) of the layer before.  Per stream every level (0 = the input) keeps rows of 4-byte
// values [rows kept][W][C]: state c (conv layers), announced value, and the deltas it emitted for
// the segment in flight.  Row r lies in slot r mod (rows kept): a ring of the rows that can still
// change or be looked at (the cone of Sec. 3), or the whole map when as many rows are kept as the
// level has.
struct EagerStep {
    Geom g;                      // unused for the input step
    int layer, n_layers;
    int o_lo, o_hi, i_lo, i_hi;
    int w_out, c_out;            // input step: shape of an input row
    int init_bias;               // the state starts from the bias (first pass of a sample)
    int fresh_lo;                // rows >= fresh_lo of this level are reached for the first time: state and
                                 // announced value start from zero whatever their slots hold
    int in_hi;                   // rows >= in_hi of the level before have not been reached yet: they read as zero
    int round_bf16;              // announced values are rounded to bfloat16 (events of a bfloat16 net)
    int in_rows, c_rows, ann_rows, dlt_rows;   // rows kept: of the level before (announced and deltas alike), of this level's maps
    const void *in;              // input step: pushed rows [position][rows][w][c], event type
    int64_t in_stream_stride;
    const void *dlt_in, *ann_in; // maps of the layer before
    int64_t in_map_stride;       // elements per stream of those
    void *c, *ann, *dlt_out;     // this layer's maps
    int64_t c_stride, ann_stride, dlt_stride;   // elements per stream
    const void *w, *bias;
    unsigned long long *stats;
};

// Steps of the gathering matrix-core kernel (k_conv_gather.hip): rows of one layer to form, or the caller's rows to take in.
constexpr int kGatherMax = 9;        // steps of a launch
constexpr int kGatherSegs = 16;      // buffers of the caller a launch can take rows from
constexpr int kBatchRows = 256;      // and rows
struct GatherStep {
    // (in the order a workgroup needs them: a scalar load brings 64 bytes)
    int tiles, take;             // workgroups (set by the launcher); 1: the caller's rows are taken in, 2: a max-pool
    int n_ct, n_pt, spt_log;     // tiles of channels; of positions per stream or group of streams; streams per tile (log2)
    int wide, n_cg;              // (set by the launcher) tiles are two by two, or their windows go through LDS; of channels then
    unsigned ct_rcp;
    int n_rows, y0;              // output rows (take: input rows): how many, first within its sample
    int n_ks, cells;             // K-steps; cells of 16 bytes per position (channels padded)
    unsigned cells_rcp;
    int slot0, ring_rows;        // ring slot of the first row of the first window (take: of row y0); rows of the ring
    int k_h, s_h_log;

    int64_t ring_stride, dst_stride;       // elements per stream
    void *ring, *dst;
    const void *w_frag, *bias;
    int h_in, p_h;
    int dst_slot0, dst_rows;     // ring slot of the first row that leaves, rows of that ring (take: first column given, columns given)

    int c_in, c_out, dst_cells, to_output;
    int act, shr, clamp_hi, layer;
    // the layer behind, whose events the emitted values are
    int next_layer, next_c_out, nk_h, ns_h_log, np_h, nh_out;
    int h_out, flat;             // flat: one position per row and kernel column (1-D)
    // rows of many positions
    int k_w, s_w_log, p_w, w_in, w_out, nk_w, ns_w_log, np_w, nw_out;
    unsigned win_rcp, wout_rcp;  // of k_w * cells, of w_out: ceil(2^32 / n)
};
struct GatherHead {
    int end[8];                  // workgroups of the steps up to and with step i (the last step's own end is not needed)
    int n, n_layers;
    int sb_log, n_sb, n_sb8;     // streams in blocks of 1 << sb_log, each of which stays on an XCD (n_sb == 0: not)
    unsigned sb_rcp;
    int n_in, seg_rows, in_stride;     // the caller's buffers: how many, rows each brings; elements per stream
    unsigned long long *stats, *issued;
    const void *in[kGatherSegs];
};
template <int NS> struct GatherBatch {
    GatherHead head;
    GatherStep st[NS];
};

// The rings of a 1-D net are laid out anew, for other numbers of rows: the newest rows of streams [first, first + n) move.
struct RingMove {
    int first, n;
    int n_units;
    struct Unit {
        void *ring;
        int row_cells;           // 16-byte cells of a row
        int keep;                // rows that move
        int from_slot, from_rows, to_slot, to_rows;            // slot of the first of them, rows of the ring
    } unit[kGatherMax - 1];
};

// Eager emission of a segment through a whole net in one launch (k_eager_pass.hip): its layers in order.
constexpr int kPassMax = 16;     // conv layers at most
constexpr int kPassStages = 8;   // stages at most: a launch takes the newest push through the first, the one before it through the second, ..
constexpr int kPassGroups = 4;   // groups of four rows of a layer that a band reaches at most
struct EagerPassStep {           // a conv layer and the 2x2 pool behind it, if there is one
    // (in the order a wave needs them, and as it needs them: every instruction of a layer is issued by all sixteen waves)
    int tasks, n_ct, n_xt;       // tiles of 16 channels x 16 positions x 4 rows; of channels, of positions
    unsigned ct_rcp, xt_rcp;
    int w, c_out, co_g;          // co_g: channels from one group of lanes to the next
    int n_ksteps;
    uint32_t w_kstep, w_ky;      // bytes from one K-step, and one tap row, to the next in the packed weights
    uint32_t c_stride;           // elements per stream
    void *c;
    const void *w_frag;

    uint32_t rows_in;            // bit i: row row0 - 1 + i is in the band that arrives
    uint32_t rows_on, rows_old;  // bit i: row row0 + i of the layer is reached / has a state already
    int band0;                   // row row0 - 1, counted from the band's first
    int cells, lds_in, in_pitch, in_stride;
    int layer, emit;             // emit: differences are passed on
    int act_none, act_lo, act_hi, act_shr;     // float32: no activation; int8: one shift and two bounds serve all three kinds
    int pool, out_w;             // out_w: positions of the rows passed on

    int lds_out, out_first;      // out_first: place of row row0 (pool: of row row0 / 2) among the rows passed on (may be negative)
    int out_pitch, out_stride, out_rows;
    int out_done, out_end;       // bytes of a row passed on: from where on no lane of the tiles writes, and its length as far as it is read
    uint32_t ann_stride;         // elements per stream
    void *ann;                   // of the pool; else of a level that is kept whole, or null: whoever wants them takes f of the state
    uint32_t row_bytes;          // of a row of state
    uint32_t pool_on;            // bit i: pooled row row0 / 2 + i is looked at
    int row0;                    // first row of the first group
    int n_groups, n_in, c_in;    // groups of four rows; delta rows that arrive

    uint16_t c_slot[4 * kPassGroups];          // of each row, among those kept
    uint32_t pool_slots[kPassGroups];          // of the pooled rows, two to a word
};
struct EagerPass {
    int n, n_layers;
    int ann0_rows, ann0_slot;    // level 0
    int lds;                     // bytes (set with the layout)
    const void *in;              // pushed rows [position][rows][w][c], event type
    int64_t in_stride, ann0_stride;
    void *ann0;
    unsigned long long *stats;
    void *hand;                  // the bands from stage to stage lie at these places behind it, in units of 256 bytes
    uint32_t hand_in[kPassStages], hand_out[kPassStages];
    int parts;                   // workgroups that share a stage of one layer
    int stage0;                  // first stage of the launch; per stage its layers (none: first == end)
    uint8_t first[kPassStages], end[kPassStages];
    EagerPassStep st[kPassMax];
    const uint32_t *open;        // not null: the launch does nothing where this is zero
};
static_assert(sizeof(EagerPass) + sizeof(StreamSel) <= 4096 && sizeof(GatherBatch<kGatherMax>) + sizeof(StreamSel) <= 4096, "likewise");

// Averaging output units: rows [first_slot, first_slot + n_rows) of the output ring are added to
// the per-channel sums of each selected stream.
struct HeadAcc {
    const void *src;             // output area [stream][out_cap][w][c], 4-byte elements
    int64_t src_stream_stride;
    int64_t out_cap;
    int w, c;
    int is_int;                  // elements are int32 (else float32)
    int zero_first;              // the sums start anew with these rows
    double count;                // positions averaged once these rows are in
    double *sums, *mean;         // [stream][c] each
};

// Fully connected output units over the last layer's map: rows [first_slot, first_slot + n_rows)
// of the output ring, which are rows row0 .. of the sample, are added, weighted, to every unit.
struct HeadUnits {
    const void *src;             // output area [stream][out_cap][w][c], 4-byte elements
    int64_t src_stream_stride;
    int64_t out_cap;
    int w, c, n_units;
    int is_int;
    int zero_first;              // the units start anew (from their bias) with these rows
    int64_t row0;
    int64_t map_elems;           // out_h * w * c: weights of one unit
    const float *weights;        // [unit][out_h][w][c]
    const float *bias;           // [unit] or null
    double *values;              // [stream][unit]
};

}  // namespace idf
