// Host side of the library: network description, workspace layout, the data-independent
// row schedule of a push (which layer receives which rows, which rows become final), and the
// kernel launches.  All arithmetic of the method runs in the kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "idf.h"
#include "idf_common.h"
#include "idf_kernels.h"

using namespace idf;

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

// Workspace of idf_open_streams_static: one array per GPU, living in the library's code object
// until the process ends.  Its name is only a handle on the host side; the device address is
// asked for once per device (scratch_of) and only that pointer is ever handed to kernels, fills
// and copies.
constexpr size_t kStaticScratchBytes = (size_t)IDF_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
struct StaticScratch { unsigned char *ptr = nullptr; bool in_use = false; };
StaticScratch g_scratch[kMaxDevices];
std::mutex g_scratch_mutex;

int ev_bytes(int prec) { return prec == IDF_PREC_F32 ? 4 : prec == IDF_PREC_BF16 ? 2 : 1; }
int w_bytes(int prec) { return ev_bytes(prec); }

}  // namespace

struct idf_net {
    int precision = 0;
    int in_h = 0, in_w = 0, in_c = 0;
    std::vector<Geom> g;
    // device images: per conv layer weights [k_h][k_w][c_in][c_out] and bias [c_out] (4-byte)
    std::vector<std::vector<unsigned char>> w_img, b_img;
    // per conv layer the matrix-core kernel can serve: weights in its fragment order (else empty)
    std::vector<std::vector<unsigned char>> wm_img;
    bool finite = true;              // no weight is infinite or NaN
    int out_w = 0, out_c = 0;
    int64_t out_h = 0;
    int open_count = 0;
};

struct StreamHost {
    int64_t r = 0;            // rows of the current sample received
    int64_t out_written = 0;  // output rows completed since open/reset
    int64_t out_read = 0;     // output rows handed over
    int64_t head_done = 0;    // output rows the averaging units have taken in
    int64_t head_base = 0;    // first of the rows they average (start of the current sample)
    int x_next = 0;           // columns of the current row received (pixel segments)
    int64_t eager_rows = 0;   // eager emission: input rows of the sample last presented that the levels have seen
    int64_t sample = 0;       // whole samples received since open/reset
    uint32_t early = 0;       // layer-by-layer pushes: matrix-core units whose waiting pool row has been counted (bit per unit)
};

// A convolution on the matrix cores, with the pool fused behind it if there is one.  Its input rows lie in a
// ring of ring_rows rows per stream, row y of sample k in slot (k * rows per sample + y) mod ring_rows.
struct RowUnit {
    int l = 0, lp = 0;        // the layer, and the layer whose rows leave the unit
    bool pool = false, last = false;
    int next = -1;            // the unit that takes those rows (-1: the output area, or a layer of another kind)
    int ring_rows = 0;
    int ring_room = 0, row_elems = 0;      // gathering kernel: rows the ring has memory for (ring_rows of them are in use); elements of a row
    size_t ring_off = 0;
    int64_t ring_stride = 0;
};

// How far a stream has come in a net whose layers run side by side: per unit the input rows that have
// arrived and the rows of c that have been formed, both counted over samples since open/reset.
struct RowProg {
    int64_t in[kRowUnits + 1] = {}, out[kRowUnits + 1] = {};
    uint32_t early = 0;       // units whose waiting pool row has been counted (bit per unit)
    bool same(const RowProg &o, int n) const
    {
        return early == o.early && memcmp(in, o.in, sizeof(int64_t) * n) == 0 && memcmp(out, o.out, sizeof(int64_t) * n) == 0;
    }
};

struct ProfRec {
    int kind, layer;
    hipEvent_t a, b;
    double bytes;
};

struct idf_streams {
    int static_dev = -1;             // >= 0: the workspace is that device's static array (given back at close)
    int ev_per_step = 0;             // int8 event path (idf_set_event_path): events a tile may hold per K-step of its contraction and still go that way; 0: off
    bool use_gather = false;         // the layers are units of the gathering kernel
    bool use_cascade1d = false;      // such a net, 1-D
    bool depth_first = false;        // whose layers run one after the other within each call
    bool prof_on = false;
    std::vector<ProfRec> prof;
    std::vector<hipEvent_t> ev_pool;
    idf_net *net = nullptr;
    int B = 0, max_seg = 0;
    int64_t out_cap = 0;
    hipStream_t st = nullptr;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    std::vector<size_t> w_off, b_off, wm_off, wg_off, ring_off, held_off, transit_off;
    std::vector<int> mfma;           // per layer: 1 = matrix-core conv kernel, 2 = pool fused into the conv before it
    std::vector<int64_t> ring_stride, held_stride, transit_stride;   // elements per stream
    std::vector<int> transit_cap;                                    // rows per stream
    size_t out_off = 0, stats_off = 0, issued_off = 0, head_off = 0;
    bool count_issued = false;       // the kernels add up what they issue (an atomic per wave: switched on for measurements)
    bool head_on = false;
    int head_units = 0;              // fully connected output units (0: only the averaging units)
    char *head_units_ws = nullptr;   // caller's buffer: weights [unit][map], bias [unit], values [stream][unit]
    bool head_units_bias = false;
    int64_t out_stride = 0;
    std::vector<std::vector<unsigned char>> gather_w;      // packed weights of the gathering kernel (kept until the upload has run)
    std::vector<GatherStep> gather;             // per unit: what a step of it holds whatever the rows
    // pushes of all streams in step that wait for their launch (idf_set_push_batching)
    int batch = 1, batch_rows = 0;              // pushes per launch; rows a launch takes at most as the rings lie now
    int batch_room = 0;                         // and as they can lie at most
    int since_read = 0;                         // 1-D nets: pushes since outputs were last read
    bool read_each = false;                     // and whether that was after a single one
    int launch_rows = 0;                        // rows that arrive with a launch of 3x3 layers at most
    int held = 0, held_rows = 0;                // waiting buffers, and the rows each of them brings
    const void *held_buf[kGatherSegs];
    // Layers on the matrix-core kernel.  Where it serves the whole net (stg2d) one launch per push holds a step
    // of every unit that has rows to form, each on rows that were complete before the launch.
    std::vector<RowUnit> units;
    std::vector<int> unit_of;                   // layer -> unit (-1: none)
    bool stg2d = false;
    bool prog_same = true;                      // all streams stand at prog_all (else each at its own)
    RowProg prog_all;
    std::vector<RowProg> prog;
    std::vector<std::pair<int, int>> push_members;   // (position, id) of the streams of the push being checked
    // eager emission: per stream and level (0 = input) rows of state, announced values and deltas in a
    // workspace of its own -- rings of the rows that can still change or be looked at (nets without
    // biases) or whole maps
    struct Eager {
        bool on = false;
        bool ring = false;
        bool one_launch = false;                  // a segment can go through the net in one launch (k_eager_pass.hip)
        bool by_stage = false;                    // but is too much for one workgroup: a launch per stage where pushes are not in stages
        char *ws = nullptr;
        std::vector<int64_t> row_elems;           // per level: W*C of one row
        std::vector<int> rows;                    // per level: rows the level has (H)
        std::vector<int> ann_rows, cd_rows;       // per level: rows kept of the announced values / of state and deltas
        std::vector<size_t> ann_off, c_off, dlt_off;   // per level (c: conv layers only)
        // Stages (eager_stages): pushes that follow one another go through the net in step, each a stage behind the next.
        // Launch number `launch` takes the push that came with launch k through stage launch - k.
        int stages = 1;
        int parts = 0;                            // workgroups of four waves that share a stage of one layer (0: a workgroup per stage)
        bool small = false;                       // workgroups of half as many waves
        int first[kPassStages + 1] = {};          // per stage its first layer
        size_t hand[kPassStages][2] = {};         // per stage where its band waits: of even and of odd launches
        int64_t launch = 0, newest = INT64_MIN / 2;       // newest: the last that brought a push
        bool on_way[kPassStages] = {};            // the push of launch k, at k mod stages, has not gone through all of them
        std::vector<EagerPass> plan;              // and what each of them does
        // Recorded into a graph (eager_flush), what is on its way may run with a replay, or not before the next call that is not recorded:
        // whichever comes first finds `open` set and clears it.  Once anything has been recorded pushes go through all layers at once.
        bool recorded = false, in_graph = false;  // a call on a recording stream; one with something on its way
        unsigned long long graph = 0;             // the recording that has it
        uint32_t *open = nullptr;
        int pays = 0;                             // pushes in a row that the stages pay for, with the launches that empty them
        int since = 0;                            // pushes since something other than pushes of all streams in step came last (eager_settle)
        int span[2] = {INT_MAX, INT_MAX};         // and how many there were before that, and before that
        std::vector<int64_t> lo, hi, seen_lo, seen_hi;
    } eager;
    // a pixel segment being pushed: columns [x_lo, x_hi) of the current row of layer 0 (else the whole row)
    struct Part { bool on = false; int x_lo = 0, x_hi = 0; bool first = true, last = true; } part;
    std::vector<StreamHost> h;
    std::vector<int> stamp;
    int stamp_gen = 0;
    idf_sizes sizes{};
};

namespace {

// Rows the last layer completes when a stream at row r receives n more rows.
int64_t output_rows_of_push(const idf_net &net, int64_t r, int n)
{
    int64_t y0 = r, cnt = n;
    for (const Geom &g : net.g) {
        int64_t a = rows_final(g, y0), b = rows_final(g, y0 + cnt);
        y0 = a;
        cnt = b - a;
        if (cnt == 0) return 0;
    }
    return cnt;
}

// Most rows a layer can emit in one step when it receives at most cap_in rows.
int max_emit(const Geom &g, int cap_in)
{
    int64_t best = 0;
    auto probe = [&](int64_t y0) {
        if (y0 < 0) return;
        int64_t cnt = cap_in;
        if (g.h_in > 0) {
            if (y0 >= g.h_in) return;
            cnt = std::min<int64_t>(cnt, g.h_in - y0);
        }
        best = std::max(best, rows_final(g, y0 + cnt) - rows_final(g, y0));
    };
    int64_t span = (int64_t)4 * g.k_h * g.s_h + cap_in + 4;
    for (int64_t y0 = 0; y0 <= span; ++y0) probe(y0);
    if (g.h_in > 0)
        for (int64_t y0 = g.h_in - span; y0 < g.h_in; ++y0) probe(y0);
    return (int)best;
}

struct Layout {
    std::vector<size_t> w_off, b_off, wm_off, wg_off, ring_off, held_off, transit_off;
    std::vector<int64_t> ring_stride, held_stride, transit_stride;
    std::vector<int> transit_cap;
    std::vector<int> mfma;           // per layer: 1 = matrix-core conv kernel, 2 = pool fused into the conv before it
    std::vector<RowUnit> units;
    size_t out_off = 0, stats_off = 0, issued_off = 0, head_off = 0, total = 0;
    int64_t out_stride = 0;
    bool gather = false;             // the gathering kernel serves this net
    bool cascade1d = false;          // and it is 1-D
    bool staged = false;             // the layers run side by side
    int launch_rows = 0, batch_rows = 0;       // rows that arrive with a launch at most: 3x3 layers, held-back pushes of a 1-D net
    idf_sizes sizes{};
};

// What gives way where a workspace does not hold the layout that is fastest.
struct Fit {
    int batch = kGatherSegs;         // 1-D nets: pushes a launch takes at most
    int launch_rows = kRowLaunchRows;          // 3x3 nets: rows that arrive with a launch at most
    bool tight = false;              // 3x3 layers: rings of the fewest rows that still move on
    bool by_kind = false;            // a net of several kinds of layers goes layer by layer (rows of c instead of twice the rows of a launch)
    bool plain = false;              // every layer on the generic kernels, which keep rows of c only
};
const Fit kFits[] = {{}, {8}, {4}, {2}, {1}, {1, 8}, {1, 4}, {1, 2}, {1, 1}, {1, 1, true}, {1, kRowLaunchRows, false, true}, {1, 1, true, true}, {1, 1, true, true, true}};

// Staged layers (one launch per push, layer l a launch behind layer l-1), rows pushed one at a time: a layer
// takes its rows in pairs, so besides the K_h rows its output rows still need at most two rows wait for it
// when a call returns.  Pushes of several rows leave up to the rows one launch completes, and one more.
constexpr int kStgWait = 2;

// Bytes a 3x3 layer's step on the gathering kernel may fetch from the caches; beyond, the net's 3x3 layers stay on the kernel
// made for them.  Measured, 32 rows through a strided layer and two 3x3 layers, here against layer by layer: 4 MB per layer and
// step 183 us against 497, 132 MB 598 against 832, 264 MB 925 against 1165 (float32); 528 MB 1570 against 1823 (bfloat16);
// 1060 MB 2977 against 2847 (float32).
constexpr double kGatherTraffic = 300e6;

// The layers run strictly depth-first within each call (nothing waits between layers across
// calls) when the staged modes are switched off.
bool strict_rows() { return getenv("IDF_NO_MFMA") || getenv("IDF_NO_ROW_STAGES"); }
bool strict_cascade() { const char *e = getenv("IDF_CASCADE_STAGES"); return e && atoi(e) <= 1; }

// Every conv layer can run on the matrix-core kernel and every pool is fused behind one.
bool net_all_mfma(const idf_net &net)
{
    const int n = (int)net.g.size();
    int units = 0;
    for (int l = 0; l < n; ++l) {
        if (net.g[l].kind == IDF_CONV) {
            if (net.wm_img[l].empty()) return false;
            ++units;
        } else if (l == 0 || net.g[l - 1].kind != IDF_CONV || net.g[l].k_w != 2) {
            return false;
        }
    }
    return units >= 1 && units <= kRowUnits;
}

// No weight is infinite or NaN.
template <class U> bool all_finite(const std::vector<unsigned char> &img, U exponent)
{
    unsigned bad = 0;
    U w[4096 / sizeof(U)];           // (of its own type and without an exit: the compiler makes vector instructions of the inner loop)
    for (size_t at = 0; at < img.size(); at += sizeof(w)) {
        const size_t n = std::min(sizeof(w), img.size() - at);
        memcpy(w, &img[at], n);
        for (size_t i = 0; i < n / sizeof(U); ++i) bad += (w[i] & exponent) == exponent;
    }
    return bad == 0;
}

// Which layers run on the matrix-core kernel: 1 = a convolution, 2 = a pool fused into the one before it.
std::vector<int> mfma_layers(const idf_net &net)
{
    std::vector<int> m(net.g.size(), 0);
    if (getenv("IDF_NO_MFMA")) return m;
    for (size_t l = 0; l < net.g.size(); ++l) {
        if (net.wm_img[l].empty()) continue;
        m[l] = 1;
        if (l + 1 < net.g.size() && net.g[l + 1].kind == IDF_MAXPOOL && net.g[l + 1].k_w == 2) m[l + 1] = 2;
    }
    return m;
}

// Rows the ring in front of layer l has on the gathering kernel when at most `rows` rows arrive with a launch: those some
// output row still needs, and those of a launch while those of the one before are being read.
int gather_ring(const Geom &g, int rows) { return 2 * rows + g.k_h + g.s_h; }

// Nets of several kinds of layers that go through the gathering kernel, all layers side by side in one launch per push.
// Layer by layer each kind has launches of its own, which is what such a net spends its time on until the layers are large.
// Then 3x3 layers are better off on the kernel made for them, which reads each weight and cell far less often.
bool gather_net(const idf_net &net, int B, int max_seg)
{
    const int n = (int)net.g.size();
    if (strict_rows() || net_all_mfma(net) || !net.finite || n > kRowUnits || max_seg > 16) return false;
    if (!net.wm_img[0].empty()) return false;       // a 3x3 layer in front has the largest map, on the kernel made for it
    int rows = max_seg;
    for (int l = 0; l < n; ++l) {
        const Geom &g = net.g[l];
        if (g.kind == IDF_MAXPOOL && (l == 0 || l == n - 1)) return false;
        if (!conv_gather_takes(net.precision, g, gather_ring(g, rows))) return false;
        rows = std::max(1, max_emit(g, rows));
        if (!net.wm_img[l].empty() && conv_gather_traffic(net.precision, g, B, rows) > kGatherTraffic) return false;
    }
    return true;
}

int make_layout(const idf_net &net, int B, int max_seg, int64_t out_cap, Layout &L, const Fit &fit = Fit())
{
    L = Layout{};
    const int n = (int)net.g.size();
    const int eb = ev_bytes(net.precision);
    size_t off = 0;
    L.w_off.assign(n, 0); L.b_off.assign(n, 0); L.wm_off.assign(n, 0); L.wg_off.assign(n, 0);
    L.ring_off.assign(n, 0); L.held_off.assign(n, 0); L.transit_off.assign(n, 0);
    L.ring_stride.assign(n, 0); L.held_stride.assign(n, 0); L.transit_stride.assign(n, 0);
    L.transit_cap.assign(n, 0);
    // rows a layer completes in one push at most, and in one launch of the staged mode
    std::vector<int> launch_cap(n, 0);
    L.launch_rows = std::min(max_seg, fit.launch_rows);
    {
        int cap = max_seg, lcap = L.launch_rows;
        for (int l = 0; l < n; ++l) {
            L.transit_cap[l] = cap = std::max(1, max_emit(net.g[l], cap));
            launch_cap[l] = lcap = std::max(1, max_emit(net.g[l], lcap));
        }
    }
    L.cascade1d = !fit.plain && cascade1d_eligible(net.precision, net.g.data(), n, max_seg);
    L.gather = L.cascade1d || (!fit.by_kind && gather_net(net, B, max_seg));
    L.mfma = L.gather || fit.plain ? std::vector<int>(n, 0) : mfma_layers(net);
    const bool staged_rows = !fit.plain && net_all_mfma(net) && !strict_rows();
    L.staged = L.gather || staged_rows;
    for (int l = 0; l < n; ++l) {
        if (net.g[l].kind != IDF_CONV) continue;
        L.w_off[l] = off; off = align_up(off + net.w_img[l].size());
        if (L.gather) { L.wg_off[l] = off; off = align_up(off + conv_gather_pack(net.precision, net.g[l], nullptr, nullptr)); }
        L.b_off[l] = off; off = align_up(off + net.b_img[l].size());
        L.wm_off[l] = off; off = align_up(off + net.wm_img[l].size());
    }
    L.sizes.weights_bytes = off;
    size_t state_per_stream = 0, transit_per_stream = 0, handover_per_stream = 0;
    for (int l = 0; l < n; ++l) {
        const Geom &g = net.g[l];
        // The retained state of a layer is K_h rows: of c, or, on the matrix cores, of the events of its input that
        // some row of c has yet to take in (they lie in the ring the layer before writes them to).
        if (g.kind == IDF_CONV) {
            L.ring_stride[l] = (int64_t)g.k_h * g.w_out * g.c_out;
            if (!L.mfma[l] && !L.gather) { L.ring_off[l] = off; off = align_up(off + (size_t)L.ring_stride[l] * 4 * B); }
            state_per_stream += (size_t)L.ring_stride[l] * 4;
            // (the method's bound; where a layer has more input than output its rows of events take more than rows of c: rows of the
            // layer before that wait)
            const int vl = conv3x3_mfma_vl(net.precision), c_in = L.gather ? (g.c_in + vl - 1) / vl * vl : g.c_in;
            const size_t events = L.mfma[l] || L.gather ? (size_t)g.k_h * g.w_in * c_in * eb : 0, rows_c = (size_t)L.ring_stride[l] * 4;
            handover_per_stream += events > rows_c ? events - rows_c : 0;
        } else {
            L.held_stride[l] = (int64_t)g.w_in * g.c_out;
            if (!L.mfma[l] && !L.gather) { L.held_off[l] = off; off = align_up(off + (size_t)L.held_stride[l] * eb * B); }
            state_per_stream += (size_t)L.held_stride[l] * eb;
        }
        if (L.mfma[l] == 1) {
            RowUnit u;
            u.l = l; u.pool = l + 1 < n && L.mfma[l + 1] == 2; u.lp = u.pool ? l + 1 : l; u.last = u.lp == n - 1;
            if (!u.last && L.mfma[u.lp + 1] == 1) u.next = (int)L.units.size() + 1;
            // rows arriving with a launch while the ones before them are being read, and the rows still needed
            const int cap = l == 0 ? max_seg : L.transit_cap[l - 1], lcap = l == 0 ? L.launch_rows : launch_cap[l - 1];
            u.ring_rows = l == 0 ? lcap + 6 : std::max(2 * lcap + 4, cap + 4);
            // Layers side by side wait for room in the ring behind them: the fewest rows are the four of a pair's windows and, where
            // rows come in pairs, one more (three may wait for the fourth).  Layer by layer all rows of a push have to fit, behind the
            // two or (a pair in front of a pool not being complete) three still needed.
            if (l > 0 && staged_rows && fit.launch_rows < kRowLaunchRows) u.ring_rows = 2 * lcap + 4;
            if (fit.tight) u.ring_rows = l == 0 ? 4 : staged_rows ? 5 : cap + (u.pool ? 3 : 2);
            u.ring_stride = (int64_t)u.ring_rows * g.w_in * g.c_in;
            u.ring_off = off; off = align_up(off + (size_t)u.ring_stride * eb * B);
            if (l > 0) {
                L.transit_off[l - 1] = u.ring_off; L.transit_stride[l - 1] = u.ring_stride;
                // rows that can wait for the layer when a call returns
                if (staged_rows) handover_per_stream += (size_t)(max_seg == 1 ? kStgWait : lcap + 1) * g.w_in * g.c_in * eb;
            }
            transit_per_stream += (size_t)u.ring_stride * eb;
            L.units.push_back(u);
        }
        // (a conv layer's rows go straight into a fused pool, or into the ring of the layer behind)
        const bool into_fused_pool = l + 1 < n && L.mfma[l + 1] == 2, into_ring = l + 1 < n && L.mfma[l + 1] == 1;
        if (l < n - 1 && !L.gather && !into_fused_pool && !into_ring) {
            L.transit_stride[l] = (int64_t)L.transit_cap[l] * g.w_out * g.c_out;
            L.transit_off[l] = off; off = align_up(off + (size_t)L.transit_stride[l] * eb * B);
            transit_per_stream += (size_t)L.transit_stride[l] * eb;
        }
    }
    if (out_cap <= 0) {
        if (net.out_h <= 0) return fail(IDF_EINVAL, "an unbounded net needs out_cap_rows > 0");
        out_cap = net.out_h;
    }
    if (out_cap < L.transit_cap[n - 1])
        return fail(IDF_EINVAL, "out_cap_rows %lld is smaller than the %d rows one push can complete",
                    (long long)out_cap, L.transit_cap[n - 1]);
    L.out_stride = out_cap * net.out_w * net.out_c;
    L.out_off = off; off = align_up(off + (size_t)L.out_stride * 4 * B);
    L.stats_off = off; off = align_up(off + (size_t)B * n * 2 * sizeof(unsigned long long));
    L.issued_off = off; off = align_up(off + (size_t)B * n * sizeof(unsigned long long));
    L.head_off = off; off = align_up(off + (size_t)B * net.out_c * 2 * sizeof(double));   // sums, means
    if (L.gather) {
        // every layer's input lies in a ring, with room (1-D) for the rows of up to kGatherSegs pushes, where they are held back
        int big = L.batch_rows = L.cascade1d ? std::min(fit.batch * max_seg, kBatchRows) : max_seg, small = max_seg;
        for (int l = 0; l < n; ++l) {
            const Geom &g = net.g[l];
            RowUnit u;
            u.l = u.lp = l; u.last = l == n - 1; u.next = l + 1 < n ? l + 1 : -1;
            u.ring_rows = gather_ring(g, small);
            u.ring_room = gather_ring(g, big);
            const int vl = conv3x3_mfma_vl(net.precision);
            u.row_elems = g.w_in * ((g.c_in + vl - 1) / vl * vl);
            u.ring_stride = (int64_t)u.ring_rows * u.row_elems;
            u.ring_off = off; off = align_up(off + (size_t)u.ring_room * u.row_elems * eb * B);
            transit_per_stream += (size_t)u.ring_room * u.row_elems * eb;
            // what is alive between two pushes
            if (l < n - 1 && !(L.cascade1d && strict_cascade())) handover_per_stream += (size_t)L.transit_cap[l] * g.w_out * g.c_out * eb;
            L.units.push_back(u);
            big = std::max(1, max_emit(g, big)); small = std::max(1, max_emit(g, small));
        }
    }
    L.total = off;
    L.sizes.workspace_bytes = off;
    L.sizes.state_bytes_per_stream = state_per_stream;
    L.sizes.handover_bytes_per_stream = handover_per_stream;
    L.sizes.retained_bytes_per_stream = state_per_stream + handover_per_stream;
    L.sizes.transit_bytes_per_stream = transit_per_stream;
    L.sizes.output_bytes_per_stream = (size_t)L.out_stride * 4;
    L.sizes.out_w = net.out_w; L.sizes.out_c = net.out_c; L.sizes.out_h = net.out_h;
    return IDF_OK;
}

// The fastest layout that `bytes` hold; `need`: what one takes (the smallest, where none fits).
int fit_layout(const idf_net &net, int B, int max_seg, int64_t out_cap, size_t bytes, Layout &L, size_t &need)
{
    need = SIZE_MAX;
    for (const Fit &fit : kFits) {
        int rc = make_layout(net, B, max_seg, out_cap, L, fit);
        if (rc != IDF_OK) return rc;
        need = std::min(need, L.total);
        if (L.total <= bytes) break;
    }
    return IDF_OK;
}

int check_ids(idf_streams *s, const int32_t *ids, int n_ids)
{
    if (n_ids < 1 || n_ids > s->B) return fail(IDF_EINVAL, "n_ids %d outside [1, %d]", n_ids, s->B);
    if (!ids) return IDF_OK;
    if (++s->stamp_gen == 0x7fffffff) { std::fill(s->stamp.begin(), s->stamp.end(), 0); s->stamp_gen = 1; }
    for (int i = 0; i < n_ids; ++i) {
        if (ids[i] < 0 || ids[i] >= s->B) return fail(IDF_EINVAL, "stream id %d outside [0, %d)", ids[i], s->B);
        if (s->stamp[ids[i]] == s->stamp_gen) return fail(IDF_EINVAL, "stream id %d given twice", ids[i]);
        s->stamp[ids[i]] = s->stamp_gen;
    }
    return IDF_OK;
}

// Splits a list of (position, id) pairs into launch selections: maximal runs that are
// contiguous in both position and id go by base, the rest by value in blocks of kSelIds.
template <class F> int for_each_selection(const std::vector<std::pair<int, int>> &members, F &&f)
{
    size_t i = 0;
    while (i < members.size()) {
        size_t j = i + 1;
        while (j < members.size() && members[j].first == members[j - 1].first + 1 &&
               members[j].second == members[j - 1].second + 1 && j - i < 65535)
            ++j;
        StreamSel sel{};
        if (j - i >= 2 || members.size() - i == 1) {
            sel.n = (int)(j - i); sel.base = members[i].second; sel.pos0 = members[i].first;
            int rc = f(sel);
            if (rc != IDF_OK) return rc;
            i = j;
            continue;
        }
        // by value: positions must still be consecutive within one selection
        j = i + 1;
        while (j < members.size() && members[j].first == members[j - 1].first + 1 && j - i < (size_t)kSelIds) ++j;
        sel.n = (int)(j - i); sel.base = -1; sel.pos0 = members[i].first;
        for (size_t k = i; k < j; ++k) sel.ids[k - i] = members[k].second;
        int rc = f(sel);
        if (rc != IDF_OK) return rc;
        i = j;
    }
    return IDF_OK;
}

int dev_fail(hipError_t e, const char *what)
{
    return fail(IDF_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

// Launch context of the next kernel: plain, or with a fresh event pair while profiling.
LaunchCtx launch_ctx(idf_streams *s, int kind, double bytes, int layer = -1)
{
    LaunchCtx c;
    c.st = s->st;
    if (!s->prof_on) return c;
    hipEvent_t ev[2] = {nullptr, nullptr};
    for (int i = 0; i < 2; ++i) {
        if (!s->ev_pool.empty()) { ev[i] = s->ev_pool.back(); s->ev_pool.pop_back(); }
        else if (hipEventCreate(&ev[i]) != hipSuccess) { ev[i] = nullptr; }
    }
    if (!ev[0] || !ev[1]) {            // out of events: run this launch unprofiled
        for (int i = 0; i < 2; ++i) if (ev[i]) s->ev_pool.push_back(ev[i]);
        return c;
    }
    c.start = ev[0]; c.stop = ev[1];
    s->prof.push_back(ProfRec{kind, layer, ev[0], ev[1], bytes});
    return c;
}

// Bytes one conv step has to move by the definition of the method: the new input rows, the
// retained rows of c it continues (read) and leaves unfinished (written), the rows it emits,
// per stream; the layer's weights once.
double conv_step_bytes(const idf_net &net, const ConvStep &a, int n_streams)
{
    const int eb = ev_bytes(net.precision);
    const double row_in = (double)a.g.w_in * a.g.c_in * eb, row_out = (double)a.g.w_out * a.g.c_out;
    const int64_t old_rows = std::max<int64_t>(0, std::min(rows_touched(a.g, a.y0), a.o_hi) - a.o_lo);
    // rows handed from layer to layer are not counted: the method does not require them to
    // leave the chip
    double per_stream = (a.in_by_position ? a.cnt * row_in : 0.0) + old_rows * row_out * 4 +
                        (double)(a.o_hi - a.o_fin) * row_out * 4 +
                        (a.to_output ? (double)(a.o_fin - a.o_lo) * row_out * 4 : 0.0);
    double weights = (double)a.g.k_h * a.g.k_w * a.g.c_in * a.g.c_out * w_bytes(net.precision) + (a.bias ? a.g.c_out * 4.0 : 0.0);
    return per_stream * n_streams + weights;
}

// Quotient and remainder of counts that are nearly always small, of which a push has some sixty: by the 64-bit instruction throughout a
// push takes 0.02 us longer (us per image, four streams out of step 4516 instead of 4498).
inline int64_t quot(int64_t a, int64_t b) { return ((uint64_t)a | (uint64_t)b) >> 32 ? a / b : (int64_t)((uint32_t)a / (uint32_t)b); }
inline int64_t rest_of(int64_t a, int64_t b) { return ((uint64_t)a | (uint64_t)b) >> 32 ? a % b : (int64_t)((uint32_t)a % (uint32_t)b); }

// ---- layers on the matrix cores -------------------------------------------------------------------
// Rows counted over samples: sample * rows per sample + row.

// Rows of c of a layer that can be formed once `in` input rows have arrived.
// (a signal without end is one sample)
int64_t rows_ready(const Geom &g, int64_t in) { return g.h_in > 0 ? quot(in, g.h_in) * g.h_out + rows_final(g, rest_of(in, g.h_in)) : rows_final(g, in); }
int64_t row_in_sample(const Geom &g, int64_t o) { return g.h_out > 0 ? rest_of(o, g.h_out) : o; }
int64_t sample_end(const Geom &g, int64_t o) { return g.h_out > 0 ? (quot(o, g.h_out) + 1) * g.h_out : INT64_MAX; }
// First input row that row o of c needs.
int64_t first_needed(const Geom &g, int64_t o)
{
    return (g.h_out > 0 ? quot(o, g.h_out) * g.h_in : 0) + std::max<int64_t>(0, row_in_sample(g, o) * g.s_h - g.p_h);
}
int mod_rows(int64_t y, int64_t n) { return y >= 0 ? (int)rest_of(y, n) : (int)((y % n + n) % n); }

// How many rows leave a unit that forms rows [o, o + n) of c (all of one sample).
int64_t rows_leaving(const idf_net &net, const RowUnit &u, int64_t o, int64_t n)
{
    if (!u.pool) return n;
    const int h = net.g[u.l].h_out, hp = net.g[u.lp].h_out;
    const int64_t y = rest_of(o, h);
    return std::min<int64_t>((y + n) / 2, hp) - std::min<int64_t>(y / 2, hp);
}
// The first of them, counted over samples.
int64_t leaving_index(const idf_net &net, const RowUnit &u, int64_t o)
{
    if (!u.pool) return o;
    const int h = net.g[u.l].h_out;
    return quot(o, h) * net.g[u.lp].h_out + rest_of(o, h) / 2;
}

// Layers of more input channels never take the event path: their share of the weights would crowd the LDS of every
// workgroup of the launch for stretches too sparse to exist in practice.
constexpr int kEventChannels = 16;

// The step that forms rows [o, o + n) of c of unit k: everything but where rows that are new in this
// launch lie (y_new) and, for a layer of another kind or the output area behind it, the destination.
void row_step(idf_streams *s, int k, int64_t o, int64_t n, int n_streams, bool counted, RowStep &a, double &bytes)
{
    const idf_net &net = *s->net;
    const RowUnit &u = s->units[k];
    const Geom &g = net.g[u.l];
    const int eb = ev_bytes(net.precision), nl = (int)net.g.size();
    a = RowStep{};
    a.w = g.w_in; a.h = g.h_in; a.c_in = g.c_in; a.c_out = g.c_out;
    a.y0 = (int)(o % g.h_out); a.n_rows = (int)n;
    a.ring_rows = u.ring_rows;
    a.slot0 = mod_rows(o / g.h_out * g.h_in + a.y0 - g.p_h, u.ring_rows);
    a.y_new = 1 << 30;
    a.act = g.act; a.shr = g.shr; a.clamp_hi = g.clamp_hi;
    a.pool = u.pool; a.pool_layer = u.pool ? u.lp : -1; a.pool_emit = 1; a.pool_from = a.y0 + (counted ? 1 : 0);
    a.layer = u.l; a.n_layers = nl;
    a.next_layer = -1;
    if (u.next >= 0) { a.next_layer = s->units[u.next].l; a.next_c_out = net.g[a.next_layer].c_out; }
    a.in_ring = s->ws + u.ring_off; a.in_stride = u.ring_stride;
    a.to_output = u.last;
    if (u.last) {
        a.dst = s->ws + s->out_off; a.dst_stride = s->out_stride; a.dst_rows = (int)s->out_cap;
    } else {
        a.dst = s->ws + s->transit_off[u.lp]; a.dst_stride = s->transit_stride[u.lp];
        a.dst_rows = u.next >= 0 ? s->units[u.next].ring_rows : s->transit_cap[u.lp];
    }
    if (u.last || u.next >= 0) a.dst_slot0 = mod_rows(leaving_index(net, u, o), a.dst_rows);
    a.wfrag = s->ws + s->wm_off[u.l];
    if (const size_t ev_at = conv3x3_mfma_event_weights(net.precision, g)) {
        // Up to how many events the stretch of a row goes the event path, once the caller has switched it on: a
        // first layer of a few channels whenever the list holds them, elsewhere ev_per_step events per 32
        // elements of the contraction.
        a.w_ev = s->ws + s->wm_off[u.l] + ev_at;
        const int vl = conv3x3_mfma_vl(net.precision), steps = (3 * g.c_in + 2 * vl - 1) / (2 * vl);
        a.ev_limit = s->ev_per_step == 0 || g.c_in > kEventChannels ? 0
                     : g.c_in < vl ? conv3x3_mfma_event_cap() : std::min(conv3x3_mfma_event_cap(), steps * s->ev_per_step);
    }
    a.bias = net.b_img[u.l].empty() ? nullptr : s->ws + s->b_off[u.l];
    a.stats = (unsigned long long *)(s->ws + s->stats_off);
    a.issued = s->count_issued ? (unsigned long long *)(s->ws + s->issued_off) : nullptr;
    conv3x3_mfma_shape(net.precision, g, n_streams, s->ev_per_step > 0, 0, a);
    // Bytes the step has to move: the input rows the rows of c need (their events), the rows that leave, weights once.
    // Rows handed from layer to layer on their way out are not counted: the method does not require them to leave the chip.
    const int64_t i_lo = std::max<int64_t>(0, a.y0 - g.p_h), i_hi = std::min<int64_t>(g.h_in, a.y0 + n - g.p_h + g.k_h - 1);
    bytes += n_streams * ((double)(i_hi - i_lo) * g.w_in * g.c_in * eb +
                          (u.last ? (double)rows_leaving(net, u, o, n) * net.out_w * net.out_c * 4 : 0.0)) +
             (double)g.k_h * g.k_w * g.c_in * g.c_out * w_bytes(net.precision) + (a.bias ? g.c_out * 4.0 : 0.0);
}

// Rows [y, y + n) of a sample (counted over samples: from `at`) go into the ring of the unit that serves layer l and
// are counted as its events; save: from which of them on (index in the sample) they are needed later.
void take_step(idf_streams *s, int k, int64_t at, int64_t n, const void *dev_rows, int row_of_buffer, int n_rows, int64_t save_at, RowStep &a)
{
    const idf_net &net = *s->net;
    const RowUnit &u = s->units[k];
    const Geom &g = net.g[u.l];
    const int vl = conv3x3_mfma_vl(net.precision);
    a = RowStep{};
    a.form = kRowTake; a.tiles = (int)n;
    a.w = g.w_in; a.h = g.h_in; a.c_in = g.c_in; a.c_out = g.c_out;
    a.cells = g.c_in % vl == 0 && g.c_in >= vl ? g.c_in / vl : 0;
    a.y0 = (int)(at % g.h_in); a.n_rows = (int)n;
    a.ring_rows = u.ring_rows; a.slot0 = mod_rows(at, u.ring_rows);
    a.in_ring = s->ws + u.ring_off; a.in_stride = u.ring_stride;
    a.x_lo = 0; a.x_hi = g.w_in;
    a.layer = u.l; a.n_layers = (int)net.g.size();
    a.stats = (unsigned long long *)(s->ws + s->stats_off);
    if (!dev_rows) return;                         // rows a layer of another kind has put into the ring: only counted
    a.in_new = dev_rows;
    a.y_new = a.y0 - row_of_buffer;
    a.y_save = a.y0 + (int)std::max<int64_t>(0, save_at - at);
    a.new_stride = (int64_t)n_rows * net.in_w * net.in_c;
    if (s->part.on) {                              // a pixel segment: one row's columns [x_lo, x_hi)
        a.x_lo = s->part.x_lo; a.x_hi = s->part.x_hi; a.y_save = a.y0; a.y_new = a.y0;
        a.new_stride = (int64_t)(a.x_hi - a.x_lo) * net.in_c;
    }
}

int launch_rows(idf_streams *s, const RowBatch &b, const StreamSel &sel, double bytes, int layer);

// Steps of more tiles than a launch takes: their first rows, then the others (no step of a batch writes what one reads).
__attribute__((noinline)) int launch_rows_in_parts(idf_streams *s, const RowBatch &b, const StreamSel &sel, double bytes, int layer)
{
    RowBatch first = b, rest;
    rest.n = 0;
    for (int k = 0; k < b.n; ++k)
        if (b.st[k].tiles > kRowTilesMax && conv3x3_mfma_split(first.st[k], rest.st[rest.n])) ++rest.n;
    if (rest.n == 0) return fail(IDF_EUNSUPPORTED, "a row of more than %d tiles", kRowTilesMax);
    int rc = launch_rows(s, first, sel, bytes, layer);
    return rc != IDF_OK ? rc : launch_rows(s, rest, sel, 0, layer);
}

int launch_rows(idf_streams *s, const RowBatch &b, const StreamSel &sel, double bytes, int layer)
{
    if (b.n == 0) return IDF_OK;
    int tiles = 0;
    for (int k = 0; k < b.n; ++k) tiles = std::max(tiles, b.st[k].tiles);
    if (tiles > kRowTilesMax) return launch_rows_in_parts(s, b, sel, bytes, layer);
    hipError_t e = launch_conv3x3_mfma_rows(s->net->precision, b, sel, launch_ctx(s, kKindConvMfma, bytes, layer));
    return e == hipSuccess ? IDF_OK : dev_fail(e, "mfma conv launch");
}

// One launch for streams that all stand at p: every unit forms the rows it has the input for -- in pairs,
// which share their weights and two of four input rows; a single row only where the sample ends or, with
// flush, where a caller wants everything out -- the first unit from the n_new rows of the caller's buffer
// too.  What a unit emits waits for the next unit's step in a later launch.  q: where they stand behind the launch.
// Returns false when the ring of the first unit has no room for the new rows yet, or when there is nothing to do.
bool row_plan(idf_streams *s, const RowProg &p, RowProg &q, int n_streams, const void *dev_rows, int row0, int n_rows, int n_new, bool flush, RowBatch &b, double &bytes)
{
    const idf_net &net = *s->net;
    const int nu = (int)s->units.size();
    q = p;
    b.n = 0;
    const bool part = s->part.on && n_new > 0;
    if (n_new > 0) b.n = 1;                        // place for the step that takes them
    int busy = 0;                                  // first unit with rows it can form (without one: past the last)
    for (busy = 0; busy < nu; ++busy) {
        const RowUnit &u = s->units[busy];
        const Geom &g = net.g[u.l];
        const int64_t end = (p.out[busy] / g.h_out + 1) * g.h_out;
        int64_t n = std::min(rows_ready(g, p.in[busy]), end) - p.out[busy];
        if (p.out[busy] + n < end && u.pool) n &= ~(int64_t)1;
        if (n > 0) break;
    }
    for (int k = nu - 1; k >= 0; --k) {            // deepest first: its workgroups run longest
        const RowUnit &u = s->units[k];
        const Geom &g = net.g[u.l];
        const int64_t have = p.in[k] + (k == 0 && !part ? n_new : 0);
        const int64_t o = p.out[k], sample_end = (o / g.h_out + 1) * g.h_out;
        int64_t n = std::min(rows_ready(g, have), sample_end) - o;
        // (a single row goes alone only when no unit before this one has anything left that could complete the pair)
        if (o + n < sample_end && (u.pool || !flush || k > busy)) n &= ~(int64_t)1;
        if (u.next >= 0) {                         // room in the ring of the unit behind (as it stands before the launch)
            const RowUnit &v = s->units[u.next];
            const int64_t room = v.ring_rows - (p.in[u.next] - first_needed(net.g[v.l], p.out[u.next]));
            while (n > 0 && rows_leaving(net, u, o, n) > room) n -= n % 2 ? 1 : 2;
        }
        if (n <= 0) continue;
        if (b.n >= kRowBatchMax) continue;
        row_step(s, k, o, n, n_streams, (q.early >> k) & 1u, b.st[b.n], bytes);
        if (k == 0 && n_new > 0 && !part && p.in[0] / g.h_in == o / g.h_out) {      // (else the new rows are of the next sample)
            b.st[b.n].in_new = (const char *)dev_rows + (int64_t)row0 * net.in_w * net.in_c * ev_bytes(net.precision);
            b.st[b.n].new_stride = (int64_t)n_rows * net.in_w * net.in_c;
            b.st[b.n].y_new = (int)(p.in[0] % g.h_in);
        }
        ++b.n;
        q.early &= ~(1u << k);
        q.out[k] = o + n;
        if (u.next >= 0) q.in[u.next] += rows_leaving(net, u, o, n);
    }
    if (s->ev_per_step == 0) {                     // which tiles a step takes goes by the launch, too
        int64_t waves = 0;
        for (int i = n_new > 0; i < b.n; ++i) waves += conv3x3_mfma_wide_waves(net.precision, net.g[b.st[i].layer], n_streams, b.st[i]);
        for (int i = n_new > 0; i < b.n && waves >= kWideLaunch; ++i)
            conv3x3_mfma_shape(net.precision, net.g[b.st[i].layer], n_streams, false, waves, b.st[i]);
    }
    if (n_new > 0) {
        q.in[0] += n_new;
        const int64_t keep = first_needed(net.g[0], q.out[0]);
        // rows still needed, and those this launch reads while it writes the new ones
        if (q.in[0] - std::min(keep, first_needed(net.g[0], p.out[0])) > s->units[0].ring_rows) return false;
        take_step(s, 0, p.in[0], n_new, dev_rows, row0, n_rows, keep, b.st[0]);
        // last in dispatch order: the shortest
        std::rotate(b.st, b.st + 1, b.st + b.n);
        bytes += (double)n_streams * n_new * net.in_w * net.in_c * ev_bytes(net.precision);
    }
    return b.n > 0;
}

// Streams that stand at p receive n_rows rows (dev_rows), or (dev_rows null) everything on its way is brought through.
int row_run(idf_streams *s, const StreamSel &sel, RowProg &p, const void *dev_rows, int n_rows)
{
    RowBatch b;
    RowProg q;                                     // (p moves on once a launch is enqueued)
    int done = 0;
    for (int guard = 0;; ++guard) {
        double bytes = 0;
        const int n_new = dev_rows ? (int)std::min<int64_t>({n_rows - done, s->launch_rows, s->net->in_h - p.in[0] % s->net->in_h}) : 0;
        if (dev_rows && done == n_rows) return IDF_OK;
        bool go = row_plan(s, p, q, sel.n, dev_rows, done, n_rows, n_new, !dev_rows, b, bytes);
        const bool took = go && n_new > 0;
        if (!go && dev_rows) go = row_plan(s, p, q, sel.n, nullptr, 0, 0, 0, guard > 64, b, bytes);
        if (!go) return dev_rows ? fail(IDF_ESTATE, "internal: rows between layers do not move on") : IDF_OK;
        int rc = launch_rows(s, b, sel, bytes, -1);
        if (rc != IDF_OK) return rc;
        p = q;
        if (took) done += n_new;
    }
}

// ---- layers on the gathering kernel (k_conv_gather.hip) ---------------------------------------------------
// A signal without end: what a step says of where its rows lie in the sample matters near the beginning only.
int64_t near_start(int64_t y) { return y < 8192 ? y : 4096 + (y & 4095); }

// The step that forms rows [o, o + n) of unit k.
void gather_step(const idf_streams *s, int k, int64_t o, int64_t n, int n_streams, GatherStep &a, double &bytes)
{
    const idf_net &net = *s->net;
    const RowUnit &u = s->units[k];
    const Geom &g = net.g[u.l];
    a = s->gather[k];
    const int64_t y = row_in_sample(g, o);
    a.y0 = (int)(g.h_out > 0 ? y : near_start(y)); a.n_rows = (int)n;
    a.slot0 = mod_rows((g.h_out > 0 ? o / g.h_out * g.h_in : 0) + y * g.s_h - g.p_h, u.ring_rows);
    a.ring_rows = u.ring_rows;
    a.dst_rows = u.last ? (int)s->out_cap : s->units[u.next].ring_rows;
    a.dst_slot0 = mod_rows(o, a.dst_rows);
    conv_gather_shape(k == 0, a);
    const double eb = ev_bytes(net.precision);
    bytes += n_streams * ((double)((n - 1) * g.s_h + g.k_h) * g.w_in * g.c_in * eb + (u.last ? (double)n * net.out_w * net.out_c * 4 : 0.0)) +
             (g.kind == IDF_CONV ? (double)g.k_h * g.k_w * g.c_in * g.c_out * w_bytes(net.precision) + (a.bias ? g.c_out * 4.0 : 0.0) : 0.0);
}

// The step that takes n rows of the caller, the first of which is row `at` counted over samples: columns [x_lo, x_hi).
void gather_take(const idf_streams *s, int64_t at, int n, int x_lo, int x_hi, GatherStep &a)
{
    const RowUnit &u = s->units[0];
    const Geom &g = s->net->g[u.l];
    a = s->gather[0];
    a.take = 1;
    a.y0 = (int)(g.h_in > 0 ? at % g.h_in : near_start(at));
    a.n_rows = n; a.ring_rows = u.ring_rows; a.slot0 = mod_rows(at, u.ring_rows);
    a.dst_slot0 = x_lo; a.dst_rows = x_hi - x_lo;
    conv_gather_shape(true, a);
}

// One launch for streams that all stand at p; as row_plan, without pairs.  chain: the layers one after the other, each on
// what the ones before it emit in this launch.
bool gather_plan(const idf_streams *s, const RowProg &p, RowProg &q, int n_streams, int n_new, bool chain, GatherHead &h, GatherStep *st, double &bytes)
{
    const idf_net &net = *s->net;
    const int nu = (int)s->units.size();
    q = p;
    h.n = 0;
    auto take = [&]() {
        gather_take(s, p.in[0], n_new, s->part.on ? s->part.x_lo : 0, s->part.on ? s->part.x_hi : net.in_w, st[h.n++]);
        bytes += (double)n_streams * n_new * net.in_w * net.in_c * ev_bytes(net.precision);
    };
    if (chain && n_new > 0) { take(); q.in[0] += n_new; }
    for (int i = 0; i < nu; ++i) {
        const int k = chain ? i : nu - 1 - i;              // (side by side: the deepest first, their tiles run longest)
        const RowUnit &u = s->units[k];
        const Geom &g = net.g[u.l];
        const int64_t o = q.out[k], in = chain ? q.in[k] : p.in[k];
        int64_t n = std::min(rows_ready(g, in), sample_end(g, o)) - o;
        if (u.next >= 0) {                         // room in the ring of the unit behind (as it stands before the step)
            const RowUnit &v = s->units[u.next];
            n = std::min<int64_t>(n, v.ring_rows - ((chain ? q.in[u.next] : p.in[u.next]) - first_needed(net.g[v.l], chain ? q.out[u.next] : p.out[u.next])));
        }
        if (n <= 0) continue;
        GatherStep &a = st[h.n++];
        gather_step(s, k, o, n, n_streams, a, bytes);
        q.out[k] = o + n;
        if (u.next >= 0) q.in[u.next] += n;
    }
    if (n_new > 0) {
        if (!chain) { take(); q.in[0] += n_new; }
        // rows still needed, and those this launch reads while it writes the new ones
        const int64_t keep = std::min(first_needed(net.g[0], q.out[0]), first_needed(net.g[0], p.out[0]));
        if (q.in[0] - keep > s->units[0].ring_rows) return false;
    }
    return h.n > 0;
}

// Streams that stand at p receive the rows of n_seg buffers of seg_rows rows each (0: none), which belong to one sample;
// out: everything on its way is brought through.
int gather_run(idf_streams *s, const StreamSel &sel, RowProg &p, const void *const *bufs, int n_seg, int seg_rows, bool out)
{
    const idf_net &net = *s->net;
    GatherHead h;
    GatherStep st[kGatherMax];
    RowProg q;                                     // (p moves on once a launch is enqueued)
    h.n_layers = (int)net.g.size();
    h.stats = (unsigned long long *)(s->ws + s->stats_off);
    h.issued = s->count_issued ? (unsigned long long *)(s->ws + s->issued_off) : nullptr;
    h.n_in = n_seg; h.seg_rows = seg_rows; h.in_stride = seg_rows * (s->part.on ? s->part.x_hi - s->part.x_lo : net.in_w) * net.in_c;
    for (int i = 0; i < n_seg; ++i) h.in[i] = bufs[i];
    // What is on its way goes through in one launch, a workgroup per stream and one layer after the other, unless that is more
    // than a tile or two per layer and stream: a launch per layer, on the whole chip, is faster then (37 audio streams with 256
    // samples each on their way: 40 us against 370).
    int64_t most = n_seg * seg_rows;               // positions of one layer that wait
    for (size_t k = 0; k < s->units.size(); ++k) {
        const Geom &g = net.g[s->units[k].l];
        most = std::max(most, (rows_ready(g, p.in[k]) - p.out[k]) * g.w_out);
    }
    const bool chain = out && (s->depth_first || most <= 32);
    for (bool fresh = n_seg > 0; fresh || out;) {
        double bytes = 0;
        const bool took = fresh && gather_plan(s, p, q, sel.n, n_seg * seg_rows, chain, h, st, bytes);
        if (!took) {
            bytes = 0;
            if (!gather_plan(s, p, q, sel.n, 0, chain, h, st, bytes)) {
                if (fresh) return fail(IDF_ESTATE, "internal: rows between layers do not move on");
                break;
            }
        }
        hipError_t e = launch_conv_gather(net.precision, h, st, sel, chain, launch_ctx(s, s->use_cascade1d ? kKindCascade1d : kKindConvGather, bytes));
        if (e != hipSuccess) return dev_fail(e, "gather launch");
        p = q;
        if (took) fresh = false;
    }
    return IDF_OK;
}

// Pushes that were held back get their launch.
int gather_flush(idf_streams *s)
{
    if (s->held == 0) return IDF_OK;
    StreamSel all{};
    all.n = s->B; all.base = 0; all.pos0 = 0;
    const int64_t before = s->prog_all.in[0];
    int rc = gather_run(s, all, s->prog_all, s->held_buf, s->held, s->held_rows, s->depth_first);
    if (s->prog_all.in[0] != before) s->held = 0;
    return rc;
}

// How many rows of the rings are in use: as many as k pushes per launch need.  Nothing is on its way: of a layer's rows at most the
// K_h newest are still needed, and they move to where the rings then have them.
int gather_rings(idf_streams *s, int k)
{
    const int nu = (int)s->units.size(), eb = ev_bytes(s->net->precision);
    int rows = std::min(k * s->max_seg, s->batch_room);
    if (rows == s->batch_rows) return IDF_OK;
    const int batch_rows = rows;
    std::vector<int> ring_rows(nu);
    for (int i = 0; i < nu; ++i) {
        const Geom &g = s->net->g[s->units[i].l];
        ring_rows[i] = std::min(s->units[i].ring_room, gather_ring(g, rows));
        rows = std::max(1, max_emit(g, rows));
    }
    auto prog = [&](int id) -> const RowProg & { return s->prog_same ? s->prog_all : s->prog[id]; };
    auto move = [&](int first, int n) {
        const RowProg &p = prog(first);
        RingMove a{};
        a.first = first; a.n = n; a.n_units = nu;
        for (int i = 0; i < nu; ++i) {
            const RowUnit &u = s->units[i];
            RingMove::Unit &v = a.unit[i];
            v.ring = s->ws + u.ring_off; v.row_cells = u.row_elems * eb / 16;
            v.keep = (int)std::min<int64_t>(p.in[i], s->net->g[u.l].k_h);
            v.from_rows = u.ring_rows; v.to_rows = ring_rows[i];
            v.from_slot = mod_rows(p.in[i] - v.keep, v.from_rows); v.to_slot = mod_rows(p.in[i] - v.keep, v.to_rows);
        }
        hipError_t e = p.in[0] == 0 ? hipSuccess : launch_ring_move(a, launch_ctx(s, kKindCascade1d, 0));
        return e == hipSuccess ? (int)IDF_OK : dev_fail(e, "ring launch");
    };
    // streams that stand at the same place together, from the side the rings grow to (every ring grows, or none does)
    const bool grow = batch_rows > s->batch_rows;
    for (int done = 0; done < s->B;) {
        const int last = grow ? s->B - 1 - done : done;
        int n = 1;
        while (done + n < s->B && (s->prog_same || prog(grow ? last - n : last + n).same(prog(last), nu))) ++n;
        int rc = move(grow ? last - n + 1 : last, n);
        if (rc != IDF_OK) return rc;
        done += n;
    }
    s->batch_rows = batch_rows;
    for (int i = 0; i < nu; ++i) {
        RowUnit &u = s->units[i];
        u.ring_rows = ring_rows[i];
        u.ring_stride = (int64_t)u.ring_rows * u.row_elems;        // (close together: a few pages hold the rings of all streams)
        s->gather[i].ring_stride = u.ring_stride;
        if (i > 0) s->gather[i - 1].dst_stride = u.ring_stride;
    }
    return IDF_OK;
}

void prog_split(idf_streams *s)
{
    if (!s->prog_same) return;
    std::fill(s->prog.begin(), s->prog.end(), s->prog_all);
    s->prog_same = false;
}
void prog_join(idf_streams *s)
{
    const int nu = (int)s->units.size();
    for (size_t i = 1; i < s->prog.size(); ++i)
        if (!s->prog[i].same(s->prog[0], nu)) return;
    s->prog_all = s->prog[0];
    s->prog_same = true;
}

// Calls f(selection, progress) for the members (position, id), those that stand at the same place together.
template <class F> int for_each_prog(idf_streams *s, const std::vector<std::pair<int, int>> &members, F &&f)
{
    const int nu = (int)s->units.size();
    if (s->prog_same) {
        if ((int)members.size() == s->B && members[0] == std::make_pair(0, 0) && members.back() == std::make_pair(s->B - 1, s->B - 1)) {
            bool straight = true;
            for (int i = 0; i < s->B && straight; ++i) straight = members[i].second == i;
            if (straight) {
                StreamSel all{};
                all.n = s->B; all.base = 0; all.pos0 = 0;
                return f(all, s->prog_all);
            }
        }
        prog_split(s);
    }
    std::vector<char> taken(members.size(), 0);
    std::vector<std::pair<int, int>> group;
    for (size_t i = 0; i < members.size(); ++i) {
        if (taken[i]) continue;
        const RowProg at = s->prog[members[i].second];
        group.clear();
        for (size_t j = i; j < members.size(); ++j)
            if (!taken[j] && s->prog[members[j].second].same(at, nu)) { taken[j] = 1; group.push_back(members[j]); }
        int rc = for_each_selection(group, [&](const StreamSel &sel) {
            RowProg moved = at;
            int rc1 = f(sel, moved);
            for (int k = 0; k < sel.n; ++k) s->prog[sel_stream(sel, k)] = moved;
            return rc1;
        });
        if (rc != IDF_OK) return rc;
    }
    if ((int)members.size() == s->B) prog_join(s);
    return IDF_OK;
}

std::vector<std::pair<int, int>> all_members(const idf_streams *s)
{
    std::vector<std::pair<int, int>> m(s->B);
    for (int i = 0; i < s->B; ++i) m[i] = {i, i};
    return m;
}

bool row_pending(const idf_streams *s, const RowProg &p)
{
    for (size_t k = 0; k < s->units.size(); ++k) {
        const RowUnit &u = s->units[k];
        const Geom &g = s->net->g[u.l];
        const int64_t o = p.out[k], end = sample_end(g, o);
        int64_t n = std::min(rows_ready(g, p.in[k]), end) - o;
        if (u.pool && o + n < end) n &= ~(int64_t)1;
        if (n > 0) return true;
    }
    return false;
}

int stg_drain(idf_streams *s)
{
    if (!s->stg2d) return IDF_OK;
    auto through = [&](const StreamSel &sel, RowProg &p) { return s->use_gather ? gather_run(s, sel, p, nullptr, 0, 1, true) : row_run(s, sel, p, nullptr, 0); };
    if (s->prog_same) {
        if (!row_pending(s, s->prog_all)) return IDF_OK;
        StreamSel all{};
        all.n = s->B; all.base = 0; all.pos0 = 0;
        return through(all, s->prog_all);
    }
    bool any = false;
    for (const RowProg &p : s->prog) any = any || row_pending(s, p);
    if (!any) return IDF_OK;
    return for_each_prog(s, all_members(s), through);
}

// Where a stream that has received `in` rows stands once nothing is on its way.
RowProg prog_at(const idf_streams *s, int64_t in, bool counted)
{
    RowProg p;
    const idf_net &net = *s->net;
    p.in[0] = in;
    for (size_t k = 0; k < s->units.size(); ++k) {
        const RowUnit &u = s->units[k];
        const Geom &g = net.g[u.l];
        int64_t o = rows_ready(g, p.in[k]);
        if (u.pool && (o % g.h_out) % 2) { --o; if (counted) p.early |= 1u << k; }
        p.out[k] = o;
        if (u.next >= 0 && g.h_out == 0) p.in[u.next] = o;
        else if (u.next >= 0) p.in[u.next] = leaving_index(net, u, o / g.h_out * g.h_out) + (u.pool ? o % g.h_out / 2 : o % g.h_out);
    }
    return p;
}

// A row of c in front of a pool whose partner has not arrived is formed with the pair.  Counters show it as
// delivered to the pool from the moment it is final: here it is formed once more, only to be counted.
int count_waiting_rows(idf_streams *s)
{
    const idf_net &net = *s->net;
    bool pool = false;
    for (const RowUnit &u : s->units) pool = pool || u.pool;
    if (!pool || s->eager.on) return IDF_OK;
    auto count = [&](const StreamSel &sel, RowProg &p) -> int {
        RowBatch b;
        b.n = 0;
        double bytes = 0;
        uint32_t early = p.early;
        for (size_t k = 0; k < s->units.size(); ++k) {
            const RowUnit &u = s->units[k];
            const Geom &g = net.g[u.l];
            if (!u.pool || ((early >> k) & 1u) || rows_ready(g, p.in[k]) <= p.out[k]) continue;
            row_step(s, (int)k, p.out[k], 1, sel.n, false, b.st[b.n], bytes);
            b.st[b.n].pool_emit = 0; b.st[b.n].issued = nullptr;
            early |= 1u << k;
            ++b.n;                                 // (units are at most kRowUnits: one launch)
        }
        int rc = launch_rows(s, b, sel, bytes, -1);
        if (rc == IDF_OK) p.early = early;
        return rc;
    };
    if (s->stg2d) return for_each_prog(s, all_members(s), count);
    for (int id = 0; id < s->B; ++id) {
        StreamHost &h = s->h[id];
        StreamSel sel{};
        sel.n = 1; sel.base = id;
        // nets with layers of other kinds run layer by layer: where unit k stands follows from the rows received
        int64_t y = h.r;
        for (size_t l = 0; l < net.g.size(); ++l) {
            const Geom &g = net.g[l];
            const int k = s->unit_of[l];
            if (k >= 0) {
                int64_t o = rows_final(g, y);
                if (s->units[k].pool && o % 2 && o < g.h_out) --o;
                RowBatch b;
                double bytes = 0;
                if (s->units[k].pool && rows_final(g, y) > o && !((h.early >> k) & 1u)) {
                    b.n = 1;
                    row_step(s, k, h.sample * g.h_out + o, 1, 1, false, b.st[0], bytes);
                    b.st[0].pool_emit = 0; b.st[0].issued = nullptr;
                    int rc = launch_rows(s, b, sel, bytes, (int)l);
                    if (rc != IDF_OK) return rc;
                    h.early |= 1u << k;
                }
            }
            y = rows_final(g, y);
        }
    }
    return IDF_OK;
}

int eager_settle(idf_streams *s);

// Everything still between stages or layers is enqueued: afterwards the work in the stream is
// that of every pushed row having gone through every layer it can influence.
int pipeline_drain(idf_streams *s)
{
    int rc = eager_settle(s);
    if (rc == IDF_OK) rc = gather_flush(s);
    return rc != IDF_OK ? rc : stg_drain(s);
}

// Layer by layer, for nets that hold layers of several kinds: streams that all stand at row r of their
// sample (`sample` whole samples before it) receive n_rows rows.
int enqueue_cascade(idf_streams *s, const StreamSel &sel, const void *dev_rows, int n_rows, int64_t r,
                    int64_t out_slot0, int64_t sample, uint32_t early)
{
    const idf_net &net = *s->net;
    const int n = (int)net.g.size();
    const int eb = ev_bytes(net.precision);
    unsigned long long *stats = (unsigned long long *)(s->ws + s->stats_off);
    const void *in = dev_rows;
    int64_t in_stride = (int64_t)n_rows * net.in_w * net.in_c;
    int64_t in_row0 = r;
    int by_pos = 1;
    int64_t y0 = r;
    int64_t cnt = n_rows;
    for (int l = 0; l < n && cnt > 0; ++l) {
        const Geom &g = net.g[l];
        const bool last = l == n - 1;
        const int64_t o_lo = rows_final(g, y0), o_fin = rows_final(g, y0 + cnt);
        void *dst = last ? (void *)(s->ws + s->out_off) : (void *)(s->ws + s->transit_off[l]);
        const int64_t dst_stride = last ? s->out_stride : s->transit_stride[l];
        if (!last && o_fin - o_lo > s->transit_cap[l])
            return fail(IDF_ESTATE, "internal: layer %d would emit %lld rows, room for %d", l,
                        (long long)(o_fin - o_lo), s->transit_cap[l]);
        // the layer behind keeps its input rows in a ring: where this layer's rows go in it
        const int dst_ring = !last && s->unit_of[l + 1] >= 0 ? s->units[s->unit_of[l + 1]].ring_rows : 0;
        const int64_t ring_slot0 = dst_ring ? mod_rows(sample * g.h_out + o_lo, dst_ring) : 0;
        if (g.kind == IDF_CONV && s->mfma[l] == 1) {
            // the rows that arrive are counted (and, when they are the caller's, kept); all rows of c they complete are formed,
            // a pool that follows taking them in pairs
            const int k = s->unit_of[l];
            const RowUnit &u = s->units[k];
            const int lp = u.lp;
            const Geom &gp = net.g[lp];
            const int64_t e_lo = u.pool ? rows_final(gp, o_lo) : o_lo, e_fin = u.pool ? rows_final(gp, o_fin) : o_fin;
            const int64_t c_lo = u.pool && o_lo < g.h_out ? o_lo & ~(int64_t)1 : o_lo;
            const int64_t c_fin = u.pool && o_fin < g.h_out ? o_fin & ~(int64_t)1 : o_fin;
            RowBatch b;
            b.n = 0;
            double bytes = 0;
            const bool own_rows = l == 0, part = own_rows && s->part.on;
            const bool counts_itself = own_rows || s->mfma[l - 1] == 0;
            if (c_fin > c_lo && !part) {
                RowStep &a = b.st[b.n++];
                row_step(s, k, sample * g.h_out + c_lo, c_fin - c_lo, sel.n, (early >> k) & 1u, a, bytes);
                if (own_rows) { a.in_new = dev_rows; a.new_stride = in_stride; a.y_new = (int)y0; }
                if (!u.last && u.next < 0) a.dst_slot0 = 0;
                if (u.last) a.dst_slot0 = (int)out_slot0;
            }
            int rc = IDF_OK;
            if (own_rows && b.n > 0 && y0 + cnt - first_needed(g, c_lo) > u.ring_rows) {
                // more rows than the ring has slots: those that are read from it go out before new ones are written to it
                rc = launch_rows(s, b, sel, bytes, l);
                if (rc != IDF_OK) return rc;
                b.n = 0; bytes = 0;
            }
            if (counts_itself)
                take_step(s, k, sample * g.h_in + y0, cnt, own_rows ? dev_rows : nullptr, 0, n_rows,
                          sample * g.h_in + (c_fin < g.h_out ? first_needed(g, c_fin) : g.h_in), b.st[b.n++]);
            rc = launch_rows(s, b, sel, bytes, l);
            if (rc != IDF_OK) return rc;
            if (c_fin > c_lo && part) {           // the row is whole only with the segment just taken: formed from the ring
                b.n = 1;
                bytes = 0;
                row_step(s, k, sample * g.h_out + c_lo, c_fin - c_lo, sel.n, (early >> k) & 1u, b.st[0], bytes);
                if (!u.last && u.next < 0) b.st[0].dst_slot0 = 0;
                if (u.last) b.st[0].dst_slot0 = (int)out_slot0;
                rc = launch_rows(s, b, sel, bytes, l);
                if (rc != IDF_OK) return rc;
            }
            in = u.last ? (void *)(s->ws + s->out_off) : (void *)(s->ws + s->transit_off[lp]);
            in_stride = u.last ? s->out_stride : s->transit_stride[lp]; in_row0 = e_lo; by_pos = 0;
            y0 = e_lo; cnt = e_fin - e_lo;
            if (u.pool) ++l;
            continue;
        } else if (g.kind == IDF_CONV) {
            const int max_rows = conv_generic_max_rows(g.c_out);
            int64_t yy = y0;
            while (yy < y0 + cnt) {
                int64_t c = y0 + cnt - yy;
                auto touched = [&](int64_t cc) {
                    return std::max(rows_touched(g, yy + cc), rows_final(g, yy + cc)) - rows_final(g, yy);
                };
                while (c > 1 && touched(c) > max_rows) c = (c + 1) / 2;
                ConvStep a{};
                a.g = g; a.layer = l; a.y0 = yy; a.cnt = (int)c;
                a.o_lo = rows_final(g, yy); a.o_fin = rows_final(g, yy + c);
                a.o_hi = std::max(rows_touched(g, yy + c), a.o_fin);
                a.ring_rows = g.k_h;
                a.in = in; a.in_stream_stride = in_stride; a.in_row0 = in_row0; a.in_by_position = by_pos;
                a.ring = s->ws + s->ring_off[l]; a.ring_stream_stride = s->ring_stride[l];
                a.dst = dst; a.dst_stream_stride = dst_stride; a.dst_row0 = o_lo; a.dst_slot0 = last ? out_slot0 : ring_slot0;
                a.dst_ring = dst_ring;
                a.to_output = last; a.out_cap = s->out_cap;
                a.w = s->ws + s->w_off[l];
                a.bias = net.b_img[l].empty() ? nullptr : s->ws + s->b_off[l];
                a.stats = stats; a.n_layers = n;
                if (l == 0 && s->part.on) {       // the pixel segment that completes a row (c == 1): layer 0 takes only its columns
                    a.x_lo = s->part.x_lo; a.x_hi = s->part.x_hi; a.cont = !s->part.first;
                    a.in_stream_stride = (int64_t)(s->part.x_hi - s->part.x_lo) * net.in_c;
                }
                conv_generic_plan(a);
                hipError_t e = launch_conv_generic(net.precision, a, sel,
                                                   launch_ctx(s, kKindConvGeneric, conv_step_bytes(net, a, sel.n), l));
                if (e != hipSuccess) return dev_fail(e, "conv launch");
                yy += c;
            }
        } else {
            PoolStep a{};
            a.g = g; a.layer = l; a.y0 = y0; a.cnt = (int)cnt; a.o_lo = o_lo; a.o_fin = o_fin;
            const int64_t y_last = y0 + cnt - 1;
            a.hold_new = (y_last % 2 == 0) && (g.h_out == 0 || y_last / 2 < g.h_out);
            a.in = in; a.in_stream_stride = in_stride; a.in_row0 = in_row0; a.in_by_position = by_pos;
            a.held = s->ws + s->held_off[l]; a.held_stream_stride = s->held_stride[l];
            a.dst = dst; a.dst_stream_stride = dst_stride; a.dst_row0 = o_lo; a.dst_slot0 = last ? out_slot0 : ring_slot0;
            a.dst_ring = dst_ring;
            a.to_output = last; a.out_cap = s->out_cap;
            a.stats = stats; a.n_layers = n;
            const double row_in = (double)g.w_in * g.c_out * eb, row_out = (double)g.w_out * g.c_out;
            const double bytes = sel.n * (cnt * row_in + (a.hold_new ? row_in : 0) + (y0 % 2 ? row_in : 0) +
                                          (double)(o_fin - o_lo) * row_out * (last ? 4 : eb));
            hipError_t e = launch_pool_generic(net.precision, a, sel, launch_ctx(s, kKindPoolGeneric, bytes, l));
            if (e != hipSuccess) return dev_fail(e, "pool launch");
        }
        in = dst; in_stride = dst_stride; in_row0 = o_lo; by_pos = 0;
        y0 = o_lo; cnt = o_fin - o_lo;
    }
    return IDF_OK;
}

// Units that have a row waiting for its partner in front of a pool after `rows` rows of the sample (layer-by-layer nets).
uint32_t early_at(const idf_streams *s, int64_t rows)
{
    uint32_t m = 0;
    for (size_t l = 0; l < s->net->g.size(); ++l) {
        const Geom &g = s->net->g[l];
        rows = rows_final(g, rows);
        const int k = s->unit_of[l];
        if (k >= 0 && s->units[k].pool && rows % 2 && rows < g.h_out) m |= 1u << k;
    }
    return m;
}

// Which of those units' waiting rows, counted before a push, still wait after it.
uint32_t early_after(const idf_streams *s, uint32_t early, int64_t before, int64_t rows)
{
    const idf_net &net = *s->net;
    int64_t a = before, b = rows;
    for (size_t l = 0; l < net.g.size(); ++l) {
        const Geom &g = net.g[l];
        const int k = s->unit_of[l];
        a = rows_final(g, a); b = rows_final(g, b);
        if (k >= 0 && s->units[k].pool && a / 2 != b / 2) early &= ~(1u << k);
        if (k >= 0 && s->units[k].pool && b >= g.h_out) early &= ~(1u << k);
    }
    return early;
}

// One stream's pieces of the workspace, in the order they are laid out in a snapshot.
template <class F> void for_each_state_piece(const idf_streams *s, int id, int64_t rows_in, F &&f)
{
    const idf_net &net = *s->net;
    const int n = (int)net.g.size();
    const int eb = ev_bytes(net.precision);
    for (int l = 0; l < n; ++l) {
        if (s->mfma[l] || s->use_gather) continue;
        if (net.g[l].kind == IDF_CONV) f(s->ring_off[l] + (size_t)id * s->ring_stride[l] * 4, (size_t)s->ring_stride[l] * 4);
        else f(s->held_off[l] + (size_t)id * s->held_stride[l] * eb, (size_t)s->held_stride[l] * eb);
    }
    if (s->use_gather) {
        // row by row, the K_h newest of every layer: how many rows of a ring are in use differs between openings
        const RowProg p = prog_at(s, rows_in, false);
        for (size_t k = 0; k < s->units.size(); ++k) {
            const RowUnit &u = s->units[k];
            const Geom &g = net.g[u.l];
            const size_t row = (size_t)u.row_elems * eb;
            for (int i = 0; i < g.k_h; ++i)
                f(u.ring_off + (size_t)id * u.ring_stride * eb + mod_rows(p.in[k] - g.k_h + i, u.ring_rows) * row, row);
        }
    } else {
        for (const RowUnit &u : s->units) f(u.ring_off + (size_t)id * u.ring_stride * eb, (size_t)u.ring_stride * eb);
    }
    f(s->stats_off + (size_t)id * n * 2 * sizeof(unsigned long long), (size_t)n * 2 * sizeof(unsigned long long));
    f(s->issued_off + (size_t)id * n * sizeof(unsigned long long), (size_t)n * sizeof(unsigned long long));
    f(s->head_off + (size_t)id * net.out_c * sizeof(double), (size_t)net.out_c * sizeof(double));
}
// The band of rows of every level that the input rows [a, b) reach: lo[lv], hi[lv] for lv = 0 ..
// n_layers (level 0 is the input itself).  With `everything` every row of every level.
void eager_bands(const idf_net &net, int64_t a, int64_t b, bool everything, std::vector<int64_t> &lo, std::vector<int64_t> &hi)
{
    const int n = (int)net.g.size();
    lo.assign(n + 1, 0); hi.assign(n + 1, 0);
    lo[0] = a; hi[0] = b;
    for (int l = 0; l < n; ++l) {
        const Geom &g = net.g[l];
        int64_t oa = 0, ob = 0;
        if (b > a) {
            if (g.kind == IDF_CONV) {
                // output rows whose footprint meets [a, b)
                const int64_t t = a + g.p_h - g.k_h + 1;
                oa = t <= 0 ? 0 : (t + g.s_h - 1) / g.s_h;
                ob = std::min<int64_t>(g.h_out, (b - 1 + g.p_h) / g.s_h + 1);
            } else {
                oa = a / 2; ob = std::min<int64_t>(g.h_out, (b - 1) / 2 + 1);
            }
            if (ob < oa) ob = oa;
        }
        if (everything) { oa = 0; ob = g.h_out; }
        lo[l + 1] = oa; hi[l + 1] = ob;
        a = oa; b = ob;
    }
}

// Layout of the eager-emission workspace for B streams pushed at most max_seg rows at a time;
// returns its size.  Nets without biases keep, per level, a ring of the rows a push can reach plus
// those a pool still looks at (every other row is final and forgotten, or still all zero); the
// last level's announced values -- the output -- are kept whole.  With biases every neuron of the
// net announces a value before any input arrives, so every level is kept whole.
size_t eager_layout(const idf_net &net, int B, int max_seg, idf_streams::Eager *e)
{
    const int n = (int)net.g.size();
    bool ring = true;
    for (int l = 0; l < n; ++l) ring = ring && net.b_img[l].empty();
    std::vector<int64_t> row_elems(n + 1);
    std::vector<int> rows(n + 1), ann_rows(n + 1), cd_rows(n + 1);
    row_elems[0] = (int64_t)net.in_w * net.in_c; rows[0] = net.in_h;
    for (int l = 0; l < n; ++l) { row_elems[l + 1] = (int64_t)net.g[l].w_out * net.g[l].c_out; rows[l + 1] = net.g[l].h_out; }
    for (int lv = 0; lv <= n; ++lv) ann_rows[lv] = cd_rows[lv] = rows[lv];
    if (ring) {
        std::vector<int64_t> need(n + 1, 1), lo, hi;
        for (int64_t a = 0; a < net.in_h; ++a) {
            eager_bands(net, a, std::min<int64_t>(a + max_seg, net.in_h), false, lo, hi);
            for (int lv = 0; lv <= n; ++lv) {
                int64_t first = lo[lv];
                // a pool re-evaluates whole windows: it also looks at the row before its band begins
                if (lv < n && net.g[lv].kind == IDF_MAXPOOL && hi[lv + 1] > lo[lv + 1]) first = std::min(first, 2 * lo[lv + 1]);
                need[lv] = std::max(need[lv], hi[lv] - first);
            }
        }
        for (int lv = 0; lv <= n; ++lv) {
            cd_rows[lv] = (int)std::min<int64_t>(rows[lv], need[lv]);
            ann_rows[lv] = lv == n ? rows[lv] : cd_rows[lv];
        }
    }
    size_t off = 0;
    std::vector<size_t> ann(n + 1), c(n + 1, 0), dlt(n + 1);
    for (int lv = 0; lv <= n; ++lv) {
        ann[lv] = off; off = align_up(off + (size_t)ann_rows[lv] * row_elems[lv] * 4 * B);
        dlt[lv] = off; off = align_up(off + (size_t)cd_rows[lv] * row_elems[lv] * 4 * B);
        if (lv > 0 && net.g[lv - 1].kind == IDF_CONV) { c[lv] = off; off = align_up(off + (size_t)cd_rows[lv] * row_elems[lv] * 4 * B); }
    }
    if (e) {
        e->ring = ring; e->row_elems = row_elems; e->rows = rows; e->ann_rows = ann_rows; e->cd_rows = cd_rows;
        e->ann_off = ann; e->c_off = c; e->dlt_off = dlt;
    }
    return off;
}

// The input rows [a, a + n_rows) through all layers in one launch; false where the bands are too large for it.
bool eager_pass_plan(const idf_streams *s, const void *dev_rows, int n_rows, int64_t a, const std::vector<int64_t> &lo,
                     const std::vector<int64_t> &hi, const std::vector<int64_t> &seen_hi, EagerPass &P, double &bytes)
{
    const idf_net &net = *s->net;
    const int n = (int)net.g.size();
    const idf_streams::Eager &E = s->eager;
    P.n = 0;
    P.n_layers = n;
    P.parts = 0;
    P.in = dev_rows; P.in_stride = (int64_t)n_rows * net.in_w * net.in_c;
    P.ann0 = E.ws + E.ann_off[0]; P.ann0_rows = E.ann_rows[0]; P.ann0_slot = (int)(a % E.ann_rows[0]);
    P.ann0_stride = (int64_t)E.ann_rows[0] * E.row_elems[0];
    P.stats = (unsigned long long *)(s->ws + s->stats_off);
    P.hand = E.ws; P.open = nullptr;
    bytes = 0;
    for (int l = 0; l < n && hi[l] > lo[l] && hi[l + 1] > lo[l + 1];) {
        const Geom &g = net.g[l];
        const int lv = l + 1;
        if (P.n == kPassMax) return false;
        EagerPassStep &L = P.st[P.n++];
        L = EagerPassStep{};
        L.layer = l;
        L.n_in = (int)(hi[l] - lo[l]);
        L.row0 = (int)(lo[lv] & ~(int64_t)1);              // (no window of a pool lies in two groups)
        L.n_groups = (int)((hi[lv] - L.row0 + 3) / 4);
        if (L.n_groups > kPassGroups) return false;
        L.band0 = L.row0 - 1 - (int)lo[l];
        L.w = g.w_out; L.c_in = g.c_in; L.c_out = g.c_out;
        const bool clamps = g.act == IDF_ACT_RELU_SHR_CLAMP;
        L.act_none = g.act == IDF_ACT_NONE; L.act_lo = L.act_none ? INT32_MIN : 0; L.act_hi = clamps ? g.clamp_hi : INT32_MAX; L.act_shr = clamps ? g.shr : 0;
        L.row_bytes = (uint32_t)E.row_elems[lv] * 4;
        // (offsets within a stream's map are 32 bits, rows of a ring 16)
        if (std::max(E.cd_rows[lv], E.ann_rows[lv]) * E.row_elems[lv] * 4 > UINT32_MAX || E.cd_rows[lv] > 1 << 16) return false;
        L.c = E.ws + E.c_off[lv]; L.c_stride = (uint32_t)(E.cd_rows[lv] * E.row_elems[lv]);
        for (int i = 0; i < 4 * L.n_groups + 2; ++i) {
            const int y = L.row0 + i;
            if (y - 1 >= lo[l] && y - 1 < hi[l]) L.rows_in |= 1u << i;
            if (i == 4 * L.n_groups) { if (y >= lo[l] && y < hi[l]) L.rows_in |= 2u << i; break; }
            if (y >= lo[lv] && y < hi[lv]) L.rows_on |= 1u << i;
            if (y < std::min(seen_hi[lv], hi[lv])) L.rows_old |= 1u << i;
            L.c_slot[i] = (uint16_t)(y % E.cd_rows[lv]);
        }
        L.ann = lv < n ? nullptr : E.ws + E.ann_off[lv];
        L.ann_stride = (uint32_t)(E.ann_rows[lv] * E.row_elems[lv]);
        L.w_frag = s->ws + s->wm_off[l];
        L.out_w = g.w_out;
        L.out_first = L.row0 - (int)lo[lv];
        bytes += (double)(hi[lv] - lo[lv]) * E.row_elems[lv] * (L.ann ? 12.0 : 8.0);
        ++l;
        if (l < n && net.g[l].kind == IDF_MAXPOOL) {
            const int pv = l + 1;
            L.pool = 1; L.out_w = net.g[l].w_out;
            if (E.ann_rows[pv] > 1 << 16 || E.ann_rows[pv] * E.row_elems[pv] * 4 > UINT32_MAX) return false;
            L.out_first = L.row0 / 2 - (int)lo[pv];
            L.ann = E.ws + E.ann_off[pv]; L.ann_stride = (uint32_t)(E.ann_rows[pv] * E.row_elems[pv]);
            for (int i = 0; i < 2 * L.n_groups; ++i) {
                const int o = L.row0 / 2 + i;
                if (o >= lo[pv] && o < hi[pv]) L.pool_on |= 1u << i;
                L.pool_slots[i / 2] |= (uint32_t)(o % E.ann_rows[pv]) << i % 2 * 16;
            }
            bytes += (double)(hi[pv] - lo[pv]) * E.row_elems[pv] * 4.0;
            ++l;
        }
        L.emit = l < n && hi[l] > lo[l] && hi[l + 1] > lo[l + 1];
    }
    return P.n > 0 && eager_pass_shape(net.precision, P);
}

// A net whose segments one launch takes through all layers: 3x3 conv layers the matrix cores serve and a 2x2 pool
// behind any of them; no biases (rings, every row starts from zero); differences that fit the operands -- a bfloat16
// net's do not, and an int8 net must clamp what it passes on.  The switches that choose between the kernels for single
// layers choose those.
constexpr int kComputeUnits = 256, kPassParts = 8, kPartsPerUnit = 4;
bool eager_one_launch(const idf_streams *s, std::vector<double> &most, bool &by_stage)
{
    most.clear();
    by_stage = false;
    const idf_net &net = *s->net;
    const bool ring = s->eager.ring;
    const int n = (int)net.g.size();
    if (!ring || net.precision == IDF_PREC_BF16 || n > 2 * kPassMax) return false;
    for (const char *e : {"IDF_EAGER_PLAIN", "IDF_EAGER_TILED", "IDF_EAGER_POS", "IDF_NO_MFMA"})
        if (getenv(e)) return false;
    for (int l = 0; l < n; ++l) {
        const Geom &g = net.g[l];
        if (g.kind == IDF_MAXPOOL) {
            if (l == 0 || net.g[l - 1].kind != IDF_CONV || g.k_w != 2 || g.s_w != 2) return false;
            continue;
        }
        if (net.wm_img[l].empty() || (l > 0 && g.c_in < 16)) return false;
        if (net.precision == IDF_PREC_I8 && l + 1 < n && g.act != IDF_ACT_RELU_SHR_CLAMP) return false;
    }
    // every segment of this opening has to go this way: announced values of conv layers are then nowhere kept but in the state
    std::vector<int64_t> lo, hi, seen_lo, seen_hi;
    EagerPass P;
    double bytes;
    for (int64_t a = 0; a < net.in_h; ++a) {
        const int64_t b = std::min<int64_t>(a + s->max_seg, net.in_h);
        eager_bands(net, a, b, false, lo, hi);
        eager_bands(net, 0, a, false, seen_lo, seen_hi);
        if (!eager_pass_plan(s, nullptr, (int)(b - a), a, lo, hi, seen_hi, P, bytes)) return false;
        // One workgroup per stream: at float32 it does 160 multiply-adds per ns, where a launch per layer takes some 14 us
        // for each layer as long as the streams are few (one stream of 32-32-64-64 channels: 57 us against about 70 at
        // 64 positions, 108 against 73 at 128; with 64 streams the two are even there).  The quantised nets are ahead
        // at any size that fits (one stream of 224 positions: 62 us against 158).  Beyond that line the nets whose layers have
        // workgroups to themselves go through in stages, or, read push by push or apart, a stage after the other (us per image, layer by layer :
        // in stages, 32-32-64-64 channels: 20 streams of 48 x 48, 2 rows per push, 1850 : 464, one stream of 48 x 128 3507 : 799, 60 of
        // 48 x 40, 3 rows, 1369 : 540; read push by push 1901 : 1029, 3595 : 2114, 1492 : 785; the first apart 34,950 : 18,789).
        double macs = 0;
        most.resize(std::max<size_t>(most.size(), P.n), 0.0);
        for (int k = 0; k < P.n; ++k) {
            const double m = 9.0 * P.st[k].n_in * 16 * P.st[k].n_xt * P.st[k].c_in * P.st[k].c_out;
            macs += m;
            most[k] = std::max(most[k], m);
        }
        by_stage = by_stage || (net.precision == IDF_PREC_F32 && s->B < 64 && macs > 160e3 * 14 * n);
    }
    const int stages = (int)most.size();
    return !by_stage || (!strict_rows() && stages >= 2 && stages <= kPassStages && stages * s->B <= kComputeUnits);
}

// How a net goes through in stages, given the multiply-adds of each of its layers in a segment and stream.  One workgroup per stream
// that takes a segment through all layers is a chain of some 3.5 us per layer on one compute unit; in stages the chain of a launch is
// as long as the longest stage, and the other compute units have work.  So there are as many stages as layers, or as compute
// units have room for a workgroup each; with more than half as many streams as compute units two stages, of workgroups of eight waves,
// two of which share a compute unit.  A stage's band waits for the next launch in memory of the workspace that layer by layer only
// needs: the announced values and differences of the level in front of it, each large enough for a band.
// Where two workgroups share a compute unit they share its SIMDs, too, and the longer stage has half the waves one workgroup would give it:
// only where that stage has no more than three fifths of the chain, or the multiply-adds of all layers take no time (1 us) beside the trips.
// us per push in one stage : two, 3-16-16-64-64 channels (0.66 to 0.70) 140 streams of 24 positions 52.5 : 58.7, 200 of 40 77.3 : 86.2; 3-64-64
// (0.80) 25.2 : 26.3; 3-16-32 (0.62) 200 of 40 12.3 : 12.8, (0.58) 256 of 24 10.7 : 10.0; int8, 16-32-64 (0.58) 14.2 : 13.8, 1-16-32-32 (0.62, few
// multiply-adds) 11.7 : 10.0.
// Measured, us per image, one stage : two : three : four (eight) of sixteen waves; two of eight waves: int8, 8 streams of 112 x 112,
// 3195 : 2117 : 1754 : 1345 (1126); 2466.  float32, 32 x 32, 64 streams 975 : 606 : 595 : 598; 597.  100 streams 994 : 631 : 851 : 871; 629.
// 128 streams 1003 : 641 : 856 : 879; 634.  200 streams 1024 : 1101 : 1181 : 1264; 943.  256 streams 1028 : 1125 : 1220 : 1319; 952.
// A stage of one layer is shared by workgroups of four waves, up to eight of them and up to four to a compute unit: its waves then have
// SIMDs to themselves, and each lane hands its differences to the next stage where the others waited for all of them in LDS first.
// us per image, one workgroup of sixteen waves : so; int8, one stream of 112 x 112 1059 : 728, eight 1128 : 776, 12 of 80 x 80 758 : 594,
// 16 of 60 x 60 492 : 428, 32 of 50 x 62 440 : 411; float32, 32 x 32, one stream 541 : 448, 16 568 : 464, 48 589 : 534, 56 and 64 593 : 601 and
// 597 : 606, 60 of 24 x 48 710 : 649.  Up to one per compute unit only: eight streams of 112 x 112 825, 12 of 80 x 80 758.  Of more streams,
// with one such workgroup to a layer: float32, 100 streams 630 : 823, 256 streams 961 : 1013.
void eager_stages(idf_streams *s, const std::vector<double> &macs)
{
    const idf_net &net = *s->net;
    idf_streams::Eager &E = s->eager;
    const int n = (int)macs.size();
    E.stages = 1; E.small = false; E.parts = 0;
    E.since = 0; E.span[0] = E.span[1] = INT_MAX;
    if (strict_rows()) return;
    int S = std::min({n, kPassStages, kComputeUnits / s->B});
    if (S < 2 && n > 1 && 2 * s->B <= 2 * kComputeUnits) { S = 2; E.small = true; }
    if (S < 2) return;
    // the division of the layers whose longest stage is shortest
    std::vector<double> sum(n + 1, 0);
    for (int k = 0; k < n; ++k) sum[k + 1] = sum[k] + 3.0 + macs[k] / (net.precision == IDF_PREC_F32 ? 350e3 : 2000e3);
    std::vector<std::vector<double>> best(S + 1, std::vector<double>(n + 1, 1e300));
    std::vector<std::vector<int>> from(S + 1, std::vector<int>(n + 1, 0));
    best[0][0] = 0;
    for (int k = 1; k <= S; ++k)
        for (int j = k; j <= n; ++j)
            for (int i = k - 1; i < j; ++i) {
                const double c = std::max(best[k - 1][i], sum[j] - sum[i]);
                if (c < best[k][j]) { best[k][j] = c; from[k][j] = i; }
            }
    if (E.small && best[S][n] > 0.6 * sum[n] && sum[n] - 3.0 * n > 1.0) return;
    for (int k = S, j = n; k >= 0; --k) { E.first[k] = j; j = from[k][j]; }
    std::vector<int> level;                                        // of each convolution
    for (size_t l = 0; l < net.g.size(); ++l)
        if (net.g[l].kind == IDF_CONV) level.push_back((int)l + 1);
    for (int k = 1; k < S; ++k) {
        const int lv = level[E.first[k] - 1];
        E.hand[k][0] = E.ann_off[lv]; E.hand[k][1] = E.dlt_off[lv];
        if (std::max(E.hand[k][0], E.hand[k][1]) / 256 > UINT32_MAX) return;
    }
    E.open = (uint32_t *)(E.ws + E.dlt_off[0]);                    // (the first stage's band is the caller's rows)
    E.stages = S;
    // Pushes in a row for which S - 1 further launches, in which stages stand empty, are made up for: us per push in one stage : in stages, read every
    // two, three, four, six, twelve pushes.  Stages of many multiply-adds: int8, 8 streams of 112 x 112 29.4 : 27.4, 29.1 : 20.7; float32, 32 x 32,
    // 64 streams 31.4 : 27.9, 31.0 : 24.5, one stream 29.7 : 26.2.  Of few: int8, 16 of 60 x 60 22.6 : 27.5, 22.3 : 20.3, 4 of 30 x 30 20.8 : 27.0,
    // 20.5 : 19.7; two stages, 4 streams of 20 positions, 7.8 : 8.8, 7.5 : 7.8, 7.3 : 7.1.  Two workgroups to a compute unit: float32, 256 of 32 x 32
    // 35.3 : 36.8, 34.2 : 34.5, 33.6 : 33.1, 33.0 : 32.0; 140 of 24 x 40, two rows, 51.7 : 56.6, 51.1 : 53.7, 50.8 : 52.3, 50.3 : 50.8, 49.9 : 49.4;
    // int8, 16-32-64 channels, 140 of 24, every four 13.2 : 14.2, six 12.2 : 12.8, twelve 11.2 : 11.2.
    if (E.small) E.pays = net.precision == IDF_PREC_F32 && sum[n] <= 32.0 ? 6 : 12;
    else E.pays = sum[n] >= 4.3 * S ? 2 : S == 2 ? 4 : 3;
    if (S == n && !E.small) E.parts = std::min(kPassParts, kPartsPerUnit * kComputeUnits / (S * s->B));
    E.plan.resize(S);
    E.launch = 0; E.newest = INT64_MIN / 2;
    std::fill(E.on_way, E.on_way + kPassStages, false);
}

// Workgroups that share a stage of one layer have its band in LDS and nothing else: as many fit a compute unit as the largest band of the
// launch leaves room for.  us per push, the LDS of the layers in one workgroup (band in, band out, of the largest layer) : so; int8, 1-32-64-64-64-64-64
// channels, 30 streams of 64 positions 32.0 : 25.0; float32, six layers of 16 channels, 17.8 : 15.3; 32-32-64-64, 60 of 48 30.6 : 29.1; most the same.
void eager_split_lds(EagerPass &a, int n_stages)
{
    a.lds = 0;
    for (int k = a.stage0; k < a.stage0 + n_stages; ++k)
        for (int j = a.first[k]; j < a.end[k]; ++j) {
            a.st[j].lds_in = 0;
            a.lds = std::max(a.lds, a.st[j].n_in * a.st[j].in_pitch);
        }
}

// The next launch of a net in stages: every push on its way goes through its next one, and a new push (planned at launch mod
// stages already) through the first.
int eager_advance(idf_streams *s, bool fresh, double bytes)
{
    idf_streams::Eager &E = s->eager;
    const int S = E.stages;
    int lo = S, hi = -1;
    EagerPass A;
    A.lds = 0;
    for (int k = 0; k < S && k <= E.launch; ++k) {
        const int64_t came = E.launch - k;
        if (k == 0 ? !fresh : !E.on_way[came % S]) continue;
        const EagerPass &P = E.plan[came % S];
        if (hi < 0) {                                              // (all but the caller's rows is the same for all pushes, and those are the first one's)
            memcpy((void *)&A, (const void *)&P, offsetof(EagerPass, st));
            memset(A.first, 0, sizeof(A.first)); memset(A.end, 0, sizeof(A.end));
            A.lds = 0; A.stage0 = lo = k; A.parts = E.parts; A.open = E.in_graph ? E.open : nullptr;
        }
        hi = k;
        const int a = E.first[k], b = std::max(a, std::min(P.n, E.first[k + 1]));
        A.first[k] = (uint8_t)a; A.end[k] = (uint8_t)b;
        A.hand_in[k] = (uint32_t)(E.hand[k][came & 1] / 256);
        A.hand_out[k] = k + 1 < S ? (uint32_t)(E.hand[k + 1][came & 1] / 256) : 0u;
        A.lds = std::max(A.lds, P.lds);
        memcpy((void *)&A.st[a], (const void *)&P.st[a], sizeof(EagerPassStep) * (size_t)(b - a));
    }
    if (hi >= 0) {
        StreamSel all{};
        all.n = s->B; all.base = 0; all.pos0 = 0;
        if (E.parts > 0) eager_split_lds(A, hi - lo + 1);
        hipError_t e = launch_eager_pass(s->net->precision, A, hi - lo + 1, E.small, all, launch_ctx(s, kKindEager, bytes, 0));
        if (e != hipSuccess) return dev_fail(e, "eager launch");
    }
    E.on_way[E.launch % S] = fresh;
    if (fresh) E.newest = E.launch;
    ++E.launch;
    return IDF_OK;
}

// 1: the stream is being recorded into a graph, as `id`; -1: it cannot be told.
int eager_recording(idf_streams *s, unsigned long long *id = nullptr)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    unsigned long long n = 0;
    if (hipStreamGetCaptureInfo(s->st, &c, &n) != hipSuccess) { (void)hipGetLastError(); return -1; }
    if (c == hipStreamCaptureStatusNone) return 0;
    s->eager.recorded = true;
    if (id) *id = n;
    return 1;
}

bool eager_pending(const idf_streams *s)
{
    const idf_streams::Eager &E = s->eager;
    return E.launch - E.newest < E.stages;
}

// Every push on its way goes through the stages that are left.  On a recording stream these launches are part of the graph, in front of what
// else is recorded, and nothing has run when the call returns: the host keeps the pushes, and until it knows better every graph and the
// next call that is not recorded bring them through.  The first that runs does it (EagerPass::open); the others find nothing left.
int eager_flush(idf_streams *s)
{
    idf_streams::Eager &E = s->eager;
    if (E.stages < 2) return IDF_OK;
    unsigned long long graph = 0;
    const bool recording = eager_recording(s, &graph) == 1;
    if (!eager_pending(s) || (recording && E.in_graph && E.graph == graph)) return IDF_OK;
    const int64_t launch = E.launch;
    bool on_way[kPassStages];
    std::copy(E.on_way, E.on_way + kPassStages, on_way);
    E.in_graph = E.in_graph || recording;
    int rc = IDF_OK;
    while (rc == IDF_OK && eager_pending(s)) rc = eager_advance(s, false, 0);
    if (rc == IDF_OK && E.in_graph) {
        hipError_t e = launch_fill_zero(E.open, 4, s->st);
        if (e != hipSuccess) rc = dev_fail(e, "eager launch");
    }
    if (recording) {
        E.launch = launch;
        std::copy(on_way, on_way + kPassStages, E.on_way);
        if (rc == IDF_OK) E.graph = graph;
    }
    return rc;
}

// Something other than the next push of all streams in step, or the end of a sample: a read, counters, a reset, a push of some streams.
int eager_settle(idf_streams *s)
{
    idf_streams::Eager &E = s->eager;
    if (E.since > 0) { E.span[1] = E.span[0]; E.span[0] = E.since; E.since = 0; }
    return eager_flush(s);
}

// One pass of eager emission for a selection of streams: the input rows [a, b) (pushed rows, or
// none when only the biases announce themselves) and, layer by layer, the band of rows they reach.
int eager_pass(idf_streams *s, const StreamSel &sel, const void *dev_rows, int n_rows, int64_t a, int64_t b, bool init_bias)
{
    const idf_net &net = *s->net;
    const int n = (int)net.g.size();
    idf_streams::Eager &E = s->eager;
    unsigned long long *stats = (unsigned long long *)(s->ws + s->stats_off);
    std::vector<int64_t> &lo = E.lo, &hi = E.hi, &seen_lo = E.seen_lo, &seen_hi = E.seen_hi;
    eager_bands(net, a, b, init_bias, lo, hi);
    eager_bands(net, 0, a, false, seen_lo, seen_hi);          // seen_hi[lv]: rows of level lv reached before this pass
    const int round_bf16 = net.precision == IDF_PREC_BF16;
    if (E.one_launch && dev_rows && !init_bias) {
        EagerPass P;
        double bytes = 0;
        if (!eager_pass_plan(s, dev_rows, n_rows, a, lo, hi, seen_hi, P, bytes)) return fail(IDF_ESTATE, "internal: a segment does not fit one launch");
        hipError_t e = hipSuccess;
        if (!E.by_stage) e = launch_eager_pass(net.precision, P, 0, false, sel, launch_ctx(s, kKindEager, bytes * sel.n, 0));
        P.parts = E.parts;
        for (int k = 0; E.by_stage && k < P.n && e == hipSuccess; ++k) {
            P.stage0 = k; P.first[k] = (uint8_t)k; P.end[k] = (uint8_t)(k + 1);
            P.hand_in[k] = (uint32_t)(E.hand[k][0] / 256); P.hand_out[k] = k + 1 < E.stages ? (uint32_t)(E.hand[k + 1][0] / 256) : 0u;
            eager_split_lds(P, 1);
            e = launch_eager_pass(net.precision, P, 1, false, sel, launch_ctx(s, kKindEager, k == 0 ? bytes * sel.n : 0.0, 0));
        }
        return e == hipSuccess ? (int)IDF_OK : dev_fail(e, "eager launch");
    }
    auto fresh_from = [&](int lv) { return E.ring ? (int)seen_hi[lv] : (int)E.rows[lv]; };    // whole maps are cleared when a sample begins
    if (dev_rows) {
        EagerStep st{};
        st.layer = 0; st.n_layers = n; st.o_lo = (int)a; st.o_hi = (int)b; st.w_out = net.in_w; st.c_out = net.in_c;
        st.in = dev_rows; st.in_stream_stride = (int64_t)n_rows * net.in_w * net.in_c;
        st.ann = E.ws + E.ann_off[0]; st.dlt_out = E.ws + E.dlt_off[0];
        st.ann_rows = E.ann_rows[0]; st.dlt_rows = E.cd_rows[0];
        st.ann_stride = (int64_t)E.ann_rows[0] * E.row_elems[0]; st.dlt_stride = (int64_t)E.cd_rows[0] * E.row_elems[0];
        st.fresh_lo = fresh_from(0);
        st.stats = stats;
        hipError_t e = launch_eager(net.precision, 0, st, sel,
                                    launch_ctx(s, kKindEager, (double)(b - a) * net.in_w * net.in_c * sel.n * 9.0, 0));
        if (e != hipSuccess) return dev_fail(e, "eager input launch");
    }
    for (int l = 0; l < n && hi[l] > lo[l]; ++l) {
        const Geom &g = net.g[l];
        if (hi[l + 1] <= lo[l + 1]) break;
        EagerStep st{};
        st.g = g; st.layer = l; st.n_layers = n; st.i_lo = (int)lo[l]; st.i_hi = (int)hi[l]; st.init_bias = init_bias;
        st.o_lo = (int)lo[l + 1]; st.o_hi = (int)hi[l + 1];
        st.fresh_lo = fresh_from(l + 1);
        st.in_hi = E.ring ? (int)hi[l] : (int)E.rows[l];
        st.round_bf16 = round_bf16 && l + 1 < n;              // the last layer's output is not rounded
        st.dlt_in = E.ws + E.dlt_off[l]; st.ann_in = E.ws + E.ann_off[l];
        st.in_rows = E.cd_rows[l];                              // (announced values of a level that feeds a layer are kept as long as its deltas)
        st.in_map_stride = (int64_t)E.cd_rows[l] * E.row_elems[l];
        st.c = g.kind == IDF_CONV ? E.ws + E.c_off[l + 1] : nullptr;
        st.ann = E.ws + E.ann_off[l + 1]; st.dlt_out = E.ws + E.dlt_off[l + 1];
        st.c_rows = st.dlt_rows = E.cd_rows[l + 1]; st.ann_rows = E.ann_rows[l + 1];
        st.c_stride = st.dlt_stride = (int64_t)E.cd_rows[l + 1] * E.row_elems[l + 1];
        st.ann_stride = (int64_t)E.ann_rows[l + 1] * E.row_elems[l + 1];
        st.w = g.kind == IDF_CONV ? s->ws + s->w_off[l] : nullptr;
        st.bias = (g.kind == IDF_CONV && !net.b_img[l].empty()) ? s->ws + s->b_off[l] : nullptr;
        st.stats = stats;
        const double cells = (double)(hi[l + 1] - lo[l + 1]) * g.w_out * g.c_out * sel.n;
        hipError_t e = launch_eager(net.precision, g.kind == IDF_CONV ? 1 : 2, st, sel,
                                    launch_ctx(s, kKindEager, cells * 16.0, l));
        if (e != hipSuccess) return dev_fail(e, "eager layer launch");
    }
    return IDF_OK;
}

// Whether a push of all streams in step goes in stages.  Begun, they go on; they begin where as many pushes as they pay for are to be expected
// before what is on its way has to be brought through: as many are left of the sample, and were made between the last two reads (the fewer of the
// two, less those made since; a row of pushes twice as long as pays ends that expectation).  Not while launches are timed (each is then the work of
// one push), and not into a graph, which may be replayed without the launches that would follow, nor behind one: a recorded read shows what
// has been pushed when it is replayed.
bool eager_staged(idf_streams *s, int n_rows)
{
    const idf_streams::Eager &E = s->eager;
    if (E.stages < 2 || E.recorded || s->prof_on) return false;
    if (!eager_pending(s)) {
        const int left = (s->net->in_h - (int)s->h[0].r + n_rows - 1) / n_rows, span = std::min(E.span[0], E.span[1]);
        const int expected = E.since < span ? span - E.since : E.since >= 2 * E.pays ? INT_MAX : 0;
        if (std::min(left, expected) < E.pays) return false;
    }
    return eager_recording(s) == 0;
}

int eager_push(idf_streams *s, const int32_t *stream_ids, int n_ids, const void *dev_rows, int n_rows)
{
    const idf_net &net = *s->net;
    const int n = (int)net.g.size();
    idf_streams::Eager &E = s->eager;
    bool in_step = n_ids == s->B;
    for (int i = 0; in_step && i < n_ids; ++i) in_step = (!stream_ids || stream_ids[i] == i) && s->h[i].r == s->h[0].r;
    const bool staged = in_step && eager_staged(s, n_rows);
    std::map<int64_t, std::vector<std::pair<int, int>>> groups;
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        const StreamHost &h = s->h[id];
        if (h.r + n_rows > net.in_h)
            return fail(IDF_ESTATE, "stream %d: rows %lld..%lld run past the sample of %d rows", id, (long long)h.r,
                        (long long)(h.r + n_rows - 1), net.in_h);
        if (!staged) groups[h.r].push_back({i, id});
    }
    const int64_t r0 = s->h[0].r;
    if (int rc = !in_step ? eager_settle(s) : !staged || r0 == 0 ? eager_flush(s) : (int)IDF_OK) return rc;
    if (staged) {
        if (r0 == 0) {                             // a sample begins: the output, which is kept whole, is zero
            hipError_t e = launch_fill_zero(E.ws + E.ann_off[n], (size_t)E.ann_rows[n] * E.row_elems[n] * 4 * s->B, s->st);
            if (e != hipSuccess) return dev_fail(e, "eager reset");
        }
        eager_bands(net, r0, r0 + n_rows, false, E.lo, E.hi);
        eager_bands(net, 0, r0, false, E.seen_lo, E.seen_hi);
        double bytes = 0;
        if (!eager_pass_plan(s, dev_rows, n_rows, r0, E.lo, E.hi, E.seen_hi, E.plan[E.launch % E.stages], bytes))
            return fail(IDF_ESTATE, "internal: a segment does not fit one launch");
        if (int rc = eager_advance(s, true, bytes * s->B)) return rc;
    }
    bool any_bias = false;
    for (int l = 0; l < n; ++l) any_bias |= !net.b_img[l].empty();
    for (auto &kv : groups) {
        const int64_t r = kv.first;
        if (r == 0) {
            // a sample begins: all state zero (Sec. 3), then the biases announce themselves.  Rings need
            // no clearing (a row starts from zero when it is first reached); what is kept whole does.
            int rc0 = for_each_selection(kv.second, [&](const StreamSel &sel) {
                // streams lie side by side in every map: one fill per map and run of streams
                for (int k = 0; k < (sel.base >= 0 ? 1 : sel.n); ++k) {
                    const int first = sel.base >= 0 ? sel.base : sel.ids[k], cnt = sel.base >= 0 ? sel.n : 1;
                    for (int lv = 0; lv <= n; ++lv) {
                        hipError_t e = hipSuccess;
                        if (!E.ring || lv == n) {
                            const size_t per = (size_t)E.ann_rows[lv] * E.row_elems[lv] * 4;
                            e = launch_fill_zero(E.ws + E.ann_off[lv] + (size_t)first * per, per * cnt, s->st);
                        }
                        if (!E.ring) {
                            const size_t per = (size_t)E.cd_rows[lv] * E.row_elems[lv] * 4, at = (size_t)first * per;
                            if (e == hipSuccess) e = launch_fill_zero(E.ws + E.dlt_off[lv] + at, per * cnt, s->st);
                            if (e == hipSuccess && lv > 0 && net.g[lv - 1].kind == IDF_CONV)
                                e = launch_fill_zero(E.ws + E.c_off[lv] + at, per * cnt, s->st);
                        }
                        if (e != hipSuccess) return dev_fail(e, "eager reset");
                    }
                }
                return (int)IDF_OK;
            });
            if (rc0 != IDF_OK) return rc0;
        }
        int rc = for_each_selection(kv.second, [&](const StreamSel &sel) {
            if (r == 0 && any_bias) {
                int rc2 = eager_pass(s, sel, nullptr, 0, 0, net.in_h, true);
                if (rc2 != IDF_OK) return rc2;
            }
            return eager_pass(s, sel, dev_rows, n_rows, r, r + n_rows, false);
        });
        if (rc != IDF_OK) return rc;
    }
    for (int i = 0; i < n_ids; ++i) {
        StreamHost &h = s->h[stream_ids ? stream_ids[i] : i];
        h.r += n_rows;
        h.eager_rows = h.r;                      // rows of the current sample the levels have seen
        if (h.r == net.in_h) h.r = 0;
    }
    if (in_step) ++E.since;
    // a whole sample waits for nothing (a launch that fails here is made again when results are asked for)
    if (staged && s->h[0].r == 0) (void)eager_flush(s);
    return IDF_OK;
}

// The averaging units take in the output rows completed since they last did.  Must run before
// read_outputs gives those rows' slots free.
int head_catch_up(idf_streams *s, const int32_t *stream_ids, int n_ids)
{
    if (!s->head_on) return IDF_OK;
    const idf_net &net = *s->net;
    struct Key { int64_t slot; int64_t n; int zero; int64_t count; int64_t row0;
                 bool operator<(const Key &o) const { return std::tie(slot, n, zero, count, row0) < std::tie(o.slot, o.n, o.zero, o.count, o.row0); } };
    std::map<Key, std::vector<std::pair<int, int>>> groups;
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        StreamHost &h = s->h[id];
        const int64_t b = h.out_written;
        int64_t a = h.head_done;
        if (b <= a) continue;
        int zero = 0;
        if (net.out_h > 0) {
            const int64_t sb = (b - 1) / net.out_h * net.out_h;      // first row of the newest sample with a row
            if (sb > h.head_base) { zero = 1; a = std::max(a, sb); h.head_base = sb; }
        }
        if (b - a > s->out_cap) return fail(IDF_ESTATE, "internal: rows for the averaging units no longer in the output area");
        if (s->head_units && a == h.head_base) zero = 1;      // first rows of a sample: the units start from their bias
        groups[Key{a % s->out_cap, b - a, zero, (b - h.head_base) * (int64_t)net.out_w, a - h.head_base}].push_back({i, id});
        h.head_done = b;
    }
    HeadAcc a{};
    a.src = s->ws + s->out_off; a.src_stream_stride = s->out_stride; a.out_cap = s->out_cap;
    a.w = net.out_w; a.c = net.out_c; a.is_int = net.precision == IDF_PREC_I8;
    a.sums = (double *)(s->ws + s->head_off); a.mean = a.sums + (size_t)s->B * net.out_c;
    for (auto &kv : groups) {
        a.zero_first = kv.first.zero; a.count = (double)kv.first.count;
        const int64_t slot = kv.first.slot;
        const int n = (int)kv.first.n;
        int rc = for_each_selection(kv.second, [&](const StreamSel &sel) {
            hipError_t e = launch_head_accumulate(a, sel, slot, n,
                                                  launch_ctx(s, kKindHead, 4.0 * n * net.out_w * net.out_c * sel.n));
            if (e == hipSuccess && s->head_units) {
                HeadUnits u{};
                u.src = a.src; u.src_stream_stride = a.src_stream_stride; u.out_cap = a.out_cap; u.w = a.w; u.c = a.c;
                u.n_units = s->head_units; u.is_int = a.is_int; u.zero_first = kv.first.zero; u.row0 = kv.first.row0;
                u.map_elems = (int64_t)net.out_h * net.out_w * net.out_c;
                u.weights = (const float *)s->head_units_ws;
                u.bias = s->head_units_bias ? u.weights + (size_t)s->head_units * u.map_elems : nullptr;
                u.values = (double *)(s->head_units_ws + align_up(((size_t)s->head_units * u.map_elems + s->head_units) * 4));
                e = launch_head_units(u, sel, slot, n, launch_ctx(s, kKindHead, 8.0 * n * net.out_w * net.out_c * sel.n * s->head_units));
            }
            return e == hipSuccess ? IDF_OK : dev_fail(e, "head launch");
        });
        if (rc != IDF_OK) return rc;
    }
    return IDF_OK;
}

int open_on(idf_net *net, int n_streams, int max_seg_rows, int64_t out_cap_rows, const Layout &L, void *dev_workspace,
            size_t workspace_bytes, void *hip_stream, idf_streams **out);

}  // namespace

// -----------------------------------------------------------------------------------------
extern "C" {

const char *idf_last_error(void) { return g_err.c_str(); }

int idf_create_net(const idf_net_desc *d, const void *const *weights, const void *const *biases,
                   idf_net **out)
{
    if (!d || !out || !d->layers) return fail(IDF_EINVAL, "null argument");
    *out = nullptr;
    if (d->precision < IDF_PREC_F32 || d->precision > IDF_PREC_I8) return fail(IDF_EINVAL, "unknown precision %d", d->precision);
    if (d->n_layers < 1 || d->n_layers > kMaxLayers) return fail(IDF_EINVAL, "n_layers %d outside [1, %d]", d->n_layers, kMaxLayers);
    if (d->in_h < 0 || d->in_w < 1 || d->in_c < 1) return fail(IDF_EINVAL, "bad input shape %d x %d x %d", d->in_h, d->in_w, d->in_c);
    idf_net *net = new (std::nothrow) idf_net;
    if (!net) return fail(IDF_ENOMEM, "out of host memory");
    net->precision = d->precision; net->in_h = d->in_h; net->in_w = d->in_w; net->in_c = d->in_c;
    int h = d->in_h, w = d->in_w, c = d->in_c;
    int rc = IDF_OK;
    for (int l = 0; l < d->n_layers && rc == IDF_OK; ++l) {
        const idf_layer &L = d->layers[l];
        Geom g{};
        g.kind = L.kind; g.c_in = L.c_in; g.c_out = L.c_out; g.k_h = L.k_h; g.k_w = L.k_w;
        g.s_h = L.s_h; g.s_w = L.s_w; g.p_h = L.p_h; g.p_w = L.p_w; g.act = L.act; g.shr = L.shr; g.clamp_hi = L.clamp_hi;
        g.h_in = h; g.w_in = w;
        if (L.kind != IDF_CONV && L.kind != IDF_MAXPOOL) rc = fail(IDF_EINVAL, "layer %d: unknown kind %d", l, L.kind);
        else if (L.c_in != c || L.c_out < 1) rc = fail(IDF_EINVAL, "layer %d: c_in %d does not follow %d channels", l, L.c_in, c);
        else if (L.k_h < 1 || L.k_w < 1 || L.s_h < 1 || L.s_w < 1 || L.p_h < 0 || L.p_w < 0) rc = fail(IDF_EINVAL, "layer %d: bad kernel/stride/padding", l);
        else if (d->in_h == 0 && L.p_h != 0) rc = fail(IDF_EINVAL, "layer %d: row padding on an unbounded stream", l);
        else if (L.kind == IDF_MAXPOOL && !(L.c_out == L.c_in && L.k_h == 2 && L.s_h == 2 && L.p_h == 0 && L.p_w == 0 &&
                                            ((L.k_w == 2 && L.s_w == 2) || (L.k_w == 1 && L.s_w == 1))))
            rc = fail(IDF_EINVAL, "layer %d: pool must be 2 x {1,2}, stride = window, no padding", l);
        else if (L.kind == IDF_CONV && (L.act < IDF_ACT_NONE || L.act > IDF_ACT_RELU_SHR_CLAMP)) rc = fail(IDF_EINVAL, "layer %d: unknown activation", l);
        else if (L.kind == IDF_CONV && (!weights || !weights[l])) rc = fail(IDF_EINVAL, "layer %d: no weights", l);
        if (rc != IDF_OK) break;
        g.h_out = d->in_h ? out_size(h, L.k_h, L.s_h, L.p_h) : 0;
        g.w_out = out_size(w, L.k_w, L.s_w, L.p_w);
        if ((d->in_h && g.h_out < 1) || g.w_out < 1) { rc = fail(IDF_EINVAL, "layer %d: window larger than its input", l); break; }
        const bool last = l == d->n_layers - 1;
        if (L.kind == IDF_CONV) {
            if (L.act == IDF_ACT_RELU_SHR_CLAMP && d->precision != IDF_PREC_I8) { rc = fail(IDF_EUNSUPPORTED, "layer %d: shift/clamp activation needs int8 precision", l); break; }
            if (L.act == IDF_ACT_RELU_SHR_CLAMP && (L.shr < 0 || L.shr > 30 || L.clamp_hi < 0 || L.clamp_hi > 127)) { rc = fail(IDF_EINVAL, "layer %d: shr/clamp_hi out of range", l); break; }
            if (d->precision == IDF_PREC_I8 && !last && L.act != IDF_ACT_RELU_SHR_CLAMP) { rc = fail(IDF_EUNSUPPORTED, "layer %d: int8 events between layers need the shift/clamp activation", l); break; }
            if (L.k_h > conv_generic_max_rows(L.c_out)) { rc = fail(IDF_EUNSUPPORTED, "layer %d: kernel height %d too large", l, L.k_h); break; }
        } else if (last && d->precision != IDF_PREC_F32) { rc = fail(IDF_EUNSUPPORTED, "a pool as the last layer needs float32 precision"); break; }
        net->g.push_back(g);
        net->w_img.emplace_back(); net->b_img.emplace_back(); net->wm_img.emplace_back();
        if (L.kind == IDF_CONV) {
            const int wb = w_bytes(d->precision);
            std::vector<unsigned char> &img = net->w_img.back();
            img.resize((size_t)L.k_h * L.k_w * L.c_in * L.c_out * wb);
            const unsigned char *src = (const unsigned char *)weights[l];
            for (int co = 0; co < L.c_out; ++co)
            for (int ci = 0; ci < L.c_in; ++ci)
            for (int ky = 0; ky < L.k_h; ++ky)
            for (int kx = 0; kx < L.k_w; ++kx) {
                size_t s_idx = (((size_t)co * L.c_in + ci) * L.k_h + ky) * L.k_w + kx;
                size_t d_idx = (((size_t)ky * L.k_w + kx) * L.c_in + ci) * L.c_out + co;
                memcpy(&img[d_idx * wb], src + s_idx * wb, wb);
            }
            if (conv3x3_mfma_eligible(d->precision, g)) {
                net->wm_img.back().resize(conv3x3_mfma_pack(d->precision, g, nullptr, nullptr));
                conv3x3_mfma_pack(d->precision, g, img.data(), net->wm_img.back().data());
            }
            if (biases && biases[l]) {
                net->b_img.back().resize((size_t)L.c_out * 4);
                memcpy(net->b_img.back().data(), biases[l], (size_t)L.c_out * 4);
            }
        }
        h = g.h_out; w = g.w_out; c = L.c_out;
    }
    if (rc != IDF_OK) { delete net; return rc; }
    net->out_h = h; net->out_w = w; net->out_c = c;
    // (asked for by gather_net alone, which nets served throughout by the 3x3 kernel never come to)
    if (net->wm_img[0].empty() && !net_all_mfma(*net))
        for (const auto &img : net->w_img)
            net->finite = net->finite && (d->precision == IDF_PREC_I8 || (d->precision == IDF_PREC_F32 ? all_finite<uint32_t>(img, 0x7f800000u) : all_finite<uint16_t>(img, 0x7f80u)));
    *out = net;
    return IDF_OK;
}

int idf_create_net_columnwise(const idf_net_desc *d, const void *const *weights, const void *const *biases,
                              idf_net **out)
{
    if (!d || !out || !d->layers) return fail(IDF_EINVAL, "null argument");
    *out = nullptr;
    if (d->n_layers < 1 || d->n_layers > kMaxLayers) return fail(IDF_EINVAL, "n_layers %d outside [1, %d]", d->n_layers, kMaxLayers);
    if (d->precision < IDF_PREC_F32 || d->precision > IDF_PREC_I8) return fail(IDF_EINVAL, "unknown precision %d", d->precision);
    // The same network with the two image axes exchanged: what streams in is then a column.
    std::vector<idf_layer> lt(d->layers, d->layers + d->n_layers);
    std::vector<std::vector<unsigned char>> wt(d->n_layers);
    std::vector<const void *> wp(d->n_layers, nullptr);
    const size_t wb = (size_t)w_bytes(d->precision);
    for (int l = 0; l < d->n_layers; ++l) {
        idf_layer &L = lt[l];
        std::swap(L.k_h, L.k_w); std::swap(L.s_h, L.s_w); std::swap(L.p_h, L.p_w);
        if (L.kind != IDF_CONV || !weights || !weights[l]) continue;
        if (L.c_in < 1 || L.c_out < 1 || L.k_h < 1 || L.k_w < 1) return fail(IDF_EINVAL, "layer %d: bad shape", l);
        // [c_out][c_in][k_h][k_w] of the image orientation -> the same with the two kernel axes exchanged
        const int kh = L.k_w, kw = L.k_h;                      // of the image orientation
        wt[l].resize((size_t)L.c_out * L.c_in * kh * kw * wb);
        const unsigned char *src = (const unsigned char *)weights[l];
        for (size_t oc = 0; oc < (size_t)L.c_out * L.c_in; ++oc)
            for (int ky = 0; ky < kh; ++ky)
                for (int kx = 0; kx < kw; ++kx)
                    memcpy(&wt[l][((oc * kw + kx) * kh + ky) * wb], src + ((oc * kh + ky) * kw + kx) * wb, wb);
        wp[l] = wt[l].data();
    }
    idf_net_desc t = *d;
    t.in_h = d->in_w; t.in_w = d->in_h; t.layers = lt.data();
    if (t.in_w < 1) return fail(IDF_EINVAL, "column-wise presentation needs the column length in_h");
    return idf_create_net(&t, wp.data(), biases, out);
}

int idf_create_net_volume(const idf_volume_desc *d, const void *const *weights, const void *const *biases, idf_net **out)
{
    if (!d || !out || !d->layers) return fail(IDF_EINVAL, "null argument");
    *out = nullptr;
    if (d->n_layers < 1 || d->n_layers > kMaxLayers) return fail(IDF_EINVAL, "n_layers %d outside [1, %d]", d->n_layers, kMaxLayers);
    if (d->precision < IDF_PREC_F32 || d->precision > IDF_PREC_I8) return fail(IDF_EINVAL, "unknown precision %d", d->precision);
    if (d->in_d < 1 || d->in_h < 1 || d->in_w < 1 || d->in_c < 1)
        return fail(IDF_EINVAL, "bad input shape %d x %d x %d x %d", d->in_d, d->in_h, d->in_w, d->in_c);
    // The column axis goes into the channels: position (row) x channel (column, c).  A layer's weights
    // become [(w_o, c_out)][(w_i, c_in)][k_d][k_h] with the entry of (w_i, w_o) taken from tap
    // kw = w_i - (w_o * s_w - p_w) where that is a tap, zero elsewhere; the bias is repeated per column.
    std::vector<idf_layer> lt(d->n_layers);
    std::vector<std::vector<unsigned char>> wt(d->n_layers), bt(d->n_layers);
    std::vector<const void *> wp(d->n_layers, nullptr), bp(d->n_layers, nullptr);
    const size_t wb = (size_t)w_bytes(d->precision);
    int w_in = d->in_w, c = d->in_c;
    for (int l = 0; l < d->n_layers; ++l) {
        const idf_volume_layer &L = d->layers[l];
        if (L.c_in != c || L.c_out < 1) return fail(IDF_EINVAL, "layer %d: c_in %d does not follow %d channels", l, L.c_in, c);
        if (L.k_d < 1 || L.k_h < 1 || L.k_w < 1 || L.s_d < 1 || L.s_h < 1 || L.s_w < 1 || L.p_d < 0 || L.p_h < 0 || L.p_w < 0)
            return fail(IDF_EINVAL, "layer %d: bad kernel/stride/padding", l);
        if (!weights || !weights[l]) return fail(IDF_EINVAL, "layer %d: no weights", l);
        const int w_out = out_size(w_in, L.k_w, L.s_w, L.p_w);
        if (w_out < 1) return fail(IDF_EINVAL, "layer %d: window larger than its input", l);
        const int64_t ci_f = (int64_t)w_in * L.c_in, co_f = (int64_t)w_out * L.c_out;
        if (ci_f > 4096 || co_f > 4096 || ci_f * co_f * L.k_d * L.k_h > ((int64_t)1 << 26))
            return fail(IDF_EUNSUPPORTED, "layer %d: %lld x %lld folded channels", l, (long long)ci_f, (long long)co_f);
        idf_layer &T = lt[l];
        T = idf_layer{};
        T.kind = IDF_CONV; T.c_in = (int)ci_f; T.c_out = (int)co_f;
        T.k_h = L.k_d; T.k_w = L.k_h; T.s_h = L.s_d; T.s_w = L.s_h; T.p_h = L.p_d; T.p_w = L.p_h;
        T.act = L.act; T.shr = L.shr; T.clamp_hi = L.clamp_hi;
        try { wt[l].assign((size_t)co_f * ci_f * L.k_d * L.k_h * wb, 0); }
        catch (const std::bad_alloc &) { return fail(IDF_ENOMEM, "out of host memory"); }
        const unsigned char *src = (const unsigned char *)weights[l];
        for (int wo = 0; wo < w_out; ++wo)
            for (int kw = 0; kw < L.k_w; ++kw) {
                const int wi = wo * L.s_w - L.p_w + kw;
                if (wi < 0 || wi >= w_in) continue;
                for (int co = 0; co < L.c_out; ++co)
                    for (int ci = 0; ci < L.c_in; ++ci)
                        for (int kd = 0; kd < L.k_d; ++kd)
                            for (int kh = 0; kh < L.k_h; ++kh) {
                                const size_t s_idx = ((((size_t)co * L.c_in + ci) * L.k_d + kd) * L.k_h + kh) * L.k_w + kw;
                                const size_t d_idx = ((((size_t)wo * L.c_out + co) * ci_f + (size_t)wi * L.c_in + ci) * L.k_d + kd) * L.k_h + kh;
                                memcpy(&wt[l][d_idx * wb], src + s_idx * wb, wb);
                            }
            }
        wp[l] = wt[l].data();
        if (biases && biases[l]) {
            bt[l].resize((size_t)co_f * 4);
            for (int wo = 0; wo < w_out; ++wo) memcpy(&bt[l][(size_t)wo * L.c_out * 4], biases[l], (size_t)L.c_out * 4);
            bp[l] = bt[l].data();
        }
        w_in = w_out; c = L.c_out;
    }
    idf_net_desc t{};
    t.precision = d->precision; t.in_h = d->in_d; t.in_w = d->in_h; t.in_c = d->in_w * d->in_c;
    t.n_layers = d->n_layers; t.layers = lt.data();
    return idf_create_net(&t, wp.data(), biases ? bp.data() : nullptr, out);
}

int idf_destroy_net(idf_net *net)
{
    if (!net) return IDF_OK;
    if (net->open_count > 0) return fail(IDF_ESTATE, "net still has %d open stream sets", net->open_count);
    delete net;
    return IDF_OK;
}

int idf_query_sizes(const idf_net *net, int n_streams, int max_seg_rows, int64_t out_cap_rows, idf_sizes *out)
{
    if (!net || !out) return fail(IDF_EINVAL, "null argument");
    if (n_streams < 1 || max_seg_rows < 1) return fail(IDF_EINVAL, "n_streams and max_seg_rows must be >= 1");
    Layout L;
    int rc = make_layout(*net, n_streams, max_seg_rows, out_cap_rows, L);
    if (rc != IDF_OK) return rc;
    *out = L.sizes;
    return IDF_OK;
}

int idf_open_streams(idf_net *net, int n_streams, int max_seg_rows, int64_t out_cap_rows, void *dev_workspace,
                     size_t workspace_bytes, void *hip_stream, idf_streams **out)
{
    if (!net || !out || !dev_workspace) return fail(IDF_EINVAL, "null argument");
    *out = nullptr;
    if (n_streams < 1 || max_seg_rows < 1) return fail(IDF_EINVAL, "n_streams and max_seg_rows must be >= 1");
    if (((uintptr_t)dev_workspace & 255) != 0) return fail(IDF_EINVAL, "workspace must be 256-byte aligned");
    Layout L;
    size_t need = 0;
    int rc = fit_layout(*net, n_streams, max_seg_rows, out_cap_rows, workspace_bytes, L, need);
    if (rc != IDF_OK) return rc;
    if (workspace_bytes < need) return fail(IDF_EINVAL, "workspace of %zu bytes, %zu needed", workspace_bytes, need);
    return open_on(net, n_streams, max_seg_rows, out_cap_rows, L, dev_workspace, workspace_bytes, hip_stream, out);
}

int idf_open_streams_static(idf_net *net, int n_streams, int max_seg_rows, int64_t out_cap_rows, void *hip_stream,
                            idf_streams **out)
{
    if (!net || !out) return fail(IDF_EINVAL, "null argument");
    *out = nullptr;
    if (n_streams < 1 || max_seg_rows < 1) return fail(IDF_EINVAL, "n_streams and max_seg_rows must be >= 1");
    Layout L;
    size_t need = 0;
    int rc = fit_layout(*net, n_streams, max_seg_rows, out_cap_rows, kStaticScratchBytes, L, need);
    if (rc != IDF_OK) return rc;
    if (need > kStaticScratchBytes)
        return fail(IDF_ENOMEM, "these streams need a workspace of %zu bytes, the static one holds %zu: fewer streams, "
                                "or idf_open_streams with a workspace of the caller's", need, kStaticScratchBytes);
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return dev_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(IDF_EDEVICE, "device %d outside the %d this library keeps a static workspace for", dev, kMaxDevices);
    unsigned char *ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        StaticScratch &sc = g_scratch[dev];
        if (!sc.ptr) {
            // this device's copy of the array: its address, asked for with the device current
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p) return dev_fail(e, "hipGetSymbolAddress(scratch)");
            sc.ptr = (unsigned char *)p;
        }
        if (sc.in_use) return fail(IDF_ESTATE, "the static workspace of device %d is taken by another set of open streams", dev);
        sc.in_use = true;
        ws = sc.ptr;
    }
    // open_on clears every byte it lays out (the array keeps what the previous streams left there)
    rc = open_on(net, n_streams, max_seg_rows, out_cap_rows, L, ws, kStaticScratchBytes, hip_stream, out);
    if (rc != IDF_OK) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        g_scratch[dev].in_use = false;
        return rc;
    }
    (*out)->static_dev = dev;
    return IDF_OK;
}

int idf_close_streams(idf_streams *s)
{
    if (!s) return IDF_OK;
    (void)pipeline_drain(s);
    hipError_t e = hipStreamSynchronize(s->st);
    for (ProfRec &r : s->prof) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    for (hipEvent_t ev : s->ev_pool) (void)hipEventDestroy(ev);
    if (s->static_dev >= 0) {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        g_scratch[s->static_dev].in_use = false;
    }
    s->net->open_count--;
    delete s;
    return e == hipSuccess ? IDF_OK : dev_fail(e, "close_streams");
}

}  // extern "C"

namespace {

// Binds n_streams streams to a workspace laid out by L: host bookkeeping, upload of the packed
// weights, every laid-out byte cleared.
int open_on(idf_net *net, int n_streams, int max_seg_rows, int64_t out_cap_rows, const Layout &L, void *dev_workspace,
            size_t workspace_bytes, void *hip_stream, idf_streams **out)
{
    idf_streams *s = new (std::nothrow) idf_streams;
    if (!s) return fail(IDF_ENOMEM, "out of host memory");
    s->net = net; s->B = n_streams; s->max_seg = max_seg_rows;
    s->out_cap = out_cap_rows > 0 ? out_cap_rows : net->out_h;
    s->st = (hipStream_t)hip_stream; s->ws = (char *)dev_workspace; s->ws_bytes = workspace_bytes;
    s->w_off = L.w_off; s->b_off = L.b_off; s->wm_off = L.wm_off; s->wg_off = L.wg_off; s->ring_off = L.ring_off; s->held_off = L.held_off;
    s->transit_off = L.transit_off; s->ring_stride = L.ring_stride; s->held_stride = L.held_stride;
    s->transit_stride = L.transit_stride; s->transit_cap = L.transit_cap;
    s->out_off = L.out_off; s->stats_off = L.stats_off; s->issued_off = L.issued_off; s->out_stride = L.out_stride; s->sizes = L.sizes;
    s->use_gather = L.gather; s->use_cascade1d = L.cascade1d; s->depth_first = L.cascade1d && strict_cascade();
    s->head_off = L.head_off;
    s->mfma = L.mfma; s->units = L.units;
    s->unit_of.assign(net->g.size(), -1);
    for (size_t k = 0; k < s->units.size(); ++k) s->unit_of[s->units[k].l] = (int)k;
    s->stg2d = L.staged; s->launch_rows = L.launch_rows; s->batch_room = L.batch_rows;
    if (s->stg2d) s->prog.assign(n_streams, RowProg{});
    if (L.gather) {
        s->batch_rows = max_seg_rows;
        for (size_t k = 0; k < s->units.size(); ++k) {
            const RowUnit &u = s->units[k];
            const Geom &g = net->g[u.l];
            GatherStep a{};
            conv_gather_layer(net->precision, g, a);
            a.layer = u.l; a.next_layer = -1;
            a.ring = s->ws + u.ring_off; a.ring_stride = u.ring_stride;
            a.to_output = u.last;
            if (u.last) {
                a.dst = s->ws + s->out_off; a.dst_stride = s->out_stride;
            } else {
                const RowUnit &v = s->units[u.next];
                const Geom &gn = net->g[v.l];
                a.dst = s->ws + v.ring_off; a.dst_stride = v.ring_stride;
                GatherStep b{};
                conv_gather_layer(net->precision, gn, b);
                a.dst_cells = b.cells;
                a.next_layer = v.l; a.next_c_out = gn.kind == IDF_CONV ? gn.c_out : 0; a.nk_h = b.k_h; a.nk_w = b.k_w; a.ns_h_log = b.s_h_log; a.ns_w_log = b.s_w_log;
                a.np_h = b.p_h; a.np_w = b.p_w; a.nh_out = b.h_out; a.nw_out = b.w_out;
            }
            a.w_frag = s->ws + s->wg_off[u.l];
            a.bias = net->b_img[u.l].empty() ? nullptr : s->ws + s->b_off[u.l];
            s->gather.push_back(a);
        }
    }
    s->h.assign(n_streams, StreamHost{});
    s->stamp.assign(n_streams, 0);
    hipError_t e = launch_fill_zero(s->ws, L.sizes.weights_bytes, s->st);     // zero padding of the weights
    for (size_t l = 0; l < net->g.size() && e == hipSuccess; ++l) {
        if (net->g[l].kind != IDF_CONV) continue;
        e = hipMemcpyAsync(s->ws + s->w_off[l], net->w_img[l].data(), net->w_img[l].size(), hipMemcpyHostToDevice, s->st);
        if (e == hipSuccess && L.gather) {
            s->gather_w.emplace_back(conv_gather_pack(net->precision, net->g[l], nullptr, nullptr));
            std::vector<unsigned char> &img = s->gather_w.back();
            conv_gather_pack(net->precision, net->g[l], net->w_img[l].data(), img.data());
            e = hipMemcpyAsync(s->ws + s->wg_off[l], img.data(), img.size(), hipMemcpyHostToDevice, s->st);
        }
        if (e == hipSuccess && !net->b_img[l].empty())
            e = hipMemcpyAsync(s->ws + s->b_off[l], net->b_img[l].data(), net->b_img[l].size(), hipMemcpyHostToDevice, s->st);
        if (e == hipSuccess && !net->wm_img[l].empty())
            e = hipMemcpyAsync(s->ws + s->wm_off[l], net->wm_img[l].data(), net->wm_img[l].size(), hipMemcpyHostToDevice, s->st);
    }
    // State needs no clearing for correctness (a row of c is initialised when first touched);
    // it is zeroed once so that the workspace never exposes stale bytes.
    if (e == hipSuccess)
        e = launch_fill_zero(s->ws + L.sizes.weights_bytes, L.total - L.sizes.weights_bytes, s->st);
    if (e != hipSuccess) { delete s; return dev_fail(e, "open_streams"); }
    net->open_count++;
    *out = s;
    return IDF_OK;
}

}  // namespace

namespace {

// n rows have gone into a stream, which complete `fresh` output rows: the host's count moves on.
inline void took_rows(const idf_streams *s, StreamHost &h, int n, int64_t fresh)
{
    const int in_h = s->net->in_h;
    h.out_written += fresh;
    if (h.early) h.early = early_after(s, h.early, h.r, h.r + n);          // (layer by layer only)
    h.r += n;
    h.x_next = 0;
    if (in_h > 0 && h.r == in_h) { h.r = 0; ++h.sample; }      // next sample
}

// A launch of a push to push_members failed.  Layers side by side: what the launches before it took in has been taken in.
__attribute__((noinline)) int push_gave_up(idf_streams *s, int rc)
{
    if (s->push_members.empty()) s->push_members = all_members(s);
    for (const auto &m : s->push_members) {
        StreamHost &h = s->h[m.second];
        const int64_t in = (s->prog_same ? s->prog_all : s->prog[m.second]).in[0] - (h.sample * s->net->in_h + h.r);
        if (in > 0) took_rows(s, h, (int)in, output_rows_of_push(*s->net, h.r, (int)in));
    }
    return rc;
}

}  // namespace

extern "C" {

int idf_push_segment(idf_streams *s, const int32_t *stream_ids, int n_ids, const void *dev_rows, int n_rows)
{
    if (!s || !dev_rows) return fail(IDF_EINVAL, "null argument");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    if (n_rows < 1 || n_rows > s->max_seg) return fail(IDF_EINVAL, "n_rows %d outside [1, %d]", n_rows, s->max_seg);
    if (s->eager.on) return eager_push(s, stream_ids, n_ids, dev_rows, n_rows);
    const idf_net &net = *s->net;
    // Validate everything before anything is enqueued.  Streams pushed in step -- the usual case --
    // share one row number and one output slot: they form one group, found without building the
    // map, and what depends on the row number only is worked out once per distinct value.
    std::vector<std::pair<int, int>> &members = s->push_members;
    members.clear();
    // (nets with layers on the matrix cores keep rows in rings by their number since open: streams there
    // go together only if they stand in the same sample too)
    typedef std::tuple<int64_t, int64_t, int64_t, uint32_t> Key;
    const bool by_sample = !s->units.empty() && !s->stg2d;
    // (layers side by side: progress is kept per stream; all streams, in step and in order, need no list: 0.02 us of a push of one
    // stream, 0.07 of 64, 0.14 of 256)
    const bool side_by_side = s->use_gather || s->stg2d;
    bool whole = side_by_side && s->prog_same && n_ids == s->B;
    for (int i = 0; whole && stream_ids && i < n_ids; ++i) whole = stream_ids[i] == i;
    Key key0{0, 0, 0, 0};
    bool one_group = true;
    int64_t memo_r = -1, memo_fresh = 0;
    auto key_of = [&](const StreamHost &h) {
        return Key{h.r, s->stg2d ? 0 : h.out_written % s->out_cap, by_sample ? h.sample : 0, by_sample ? h.early : 0};
    };
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        const StreamHost &h = s->h[id];
        if (h.x_next != 0 && !s->part.on)
            return fail(IDF_ESTATE, "stream %d: %d columns of a row were pushed as pixels, the row must be finished that way", id, h.x_next);
        if (net.in_h > 0 && h.r + n_rows > net.in_h)
            return fail(IDF_ESTATE, "stream %d: rows %lld..%lld run past the sample of %d rows", id,
                        (long long)h.r, (long long)(h.r + n_rows - 1), net.in_h);
        if (h.r != memo_r) { memo_r = h.r; memo_fresh = output_rows_of_push(net, h.r, n_rows); }
        const int64_t fresh = memo_fresh;
        if (h.out_written - h.out_read + fresh > s->out_cap)
            return fail(IDF_ESTATE, "stream %d: output area full (%lld rows waiting, %lld more would complete, room for %lld)",
                        id, (long long)(h.out_written - h.out_read), (long long)fresh, (long long)s->out_cap);
        if (!whole) members.push_back({i, id});
        if (side_by_side) continue;
        const Key key = key_of(h);
        if (i == 0) key0 = key;
        else if (key != key0) one_group = false;
    }
    // every launch of streams at the same place
    auto run = [&](auto &&f) {
        if (!whole) return for_each_prog(s, members, f);
        StreamSel all{};
        all.n = s->B; all.base = 0; all.pos0 = 0;
        return f(all, s->prog_all);
    };
    auto deliver = [&](const Key &key, const std::vector<std::pair<int, int>> &group) {
        return for_each_selection(group, [&](const StreamSel &sel) {
            return enqueue_cascade(s, sel, dev_rows, n_rows, std::get<0>(key), std::get<1>(key), std::get<2>(key), std::get<3>(key));
        });
    };
    if (s->use_cascade1d) {
        if (whole && s->batch > 1) {
            // held back until there are enough of them; a launch takes buffers of one size and of one sample
            if (s->held > 0 && (s->held_rows != n_rows || s->h[0].r == 0 || (s->held + 1) * n_rows > s->batch_rows)) rc = gather_flush(s);
            if (rc != IDF_OK) return rc;
            s->held_buf[s->held++] = dev_rows; s->held_rows = n_rows;
            if (s->held >= s->batch || (s->held + 1) * n_rows > s->batch_rows) rc = gather_flush(s);
            if (rc != IDF_OK && s->held > 0) --s->held;                      // (those before it still wait)
        } else {
            rc = gather_flush(s);
            if (rc != IDF_OK) return rc;
            // A signal that is read push by push goes through all layers with the push: what the read would bring out is out already.
            // (us per push and read, audio net, one stream with 16 samples 29.4 -> 27.7, 4 samples 28.0 -> 26.3, 64 streams 31.8 -> 29.9)
            const bool out = s->depth_first || (s->read_each && s->since_read == 0);
            rc = run([&](const StreamSel &sel, RowProg &p) { return gather_run(s, sel, p, &dev_rows, 1, n_rows, out); });
        }
        if (rc != IDF_OK) return push_gave_up(s, rc);
    } else if (s->use_gather) {
        rc = run([&](const StreamSel &sel, RowProg &p) { return gather_run(s, sel, p, &dev_rows, 1, n_rows, false); });
        if (rc != IDF_OK) return push_gave_up(s, rc);
    } else if (s->stg2d) {
        rc = run([&](const StreamSel &sel, RowProg &p) { return row_run(s, sel, p, dev_rows, n_rows); });
        if (rc != IDF_OK) return push_gave_up(s, rc);
    } else if (one_group) {
        rc = deliver(key0, members);
        if (rc != IDF_OK) return rc;
    } else {
        std::map<Key, std::vector<std::pair<int, int>>> groups;
        for (const auto &m : members) groups[key_of(s->h[m.second])].push_back(m);
        for (auto &kv : groups) {
            rc = deliver(kv.first, kv.second);
            if (rc != IDF_OK) return rc;
        }
    }
    ++s->since_read;
    memo_r = -1;
    for (int i = 0; i < n_ids; ++i) {
        StreamHost &h = s->h[stream_ids ? stream_ids[i] : i];
        if (h.r != memo_r) { memo_r = h.r; memo_fresh = output_rows_of_push(net, h.r, n_rows); }
        h.out_written += memo_fresh;
        if (by_sample && h.early) h.early = early_after(s, h.early, h.r, h.r + n_rows);
        h.r += n_rows;
        h.x_next = 0;
        if (net.in_h > 0 && h.r == net.in_h) { h.r = 0; ++h.sample; }      // next sample
    }
    return IDF_OK;
}

int idf_push_pixels(idf_streams *s, const int32_t *stream_ids, int n_ids, const void *dev_pixels, int x0, int n_px)
{
    if (!s || !dev_pixels) return fail(IDF_EINVAL, "null argument");
    const idf_net &net = *s->net;
    if (n_px < 1 || x0 < 0 || x0 + n_px > net.in_w) return fail(IDF_EINVAL, "columns %d..%d outside the row of %d", x0, x0 + n_px - 1, net.in_w);
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "pixel segments are not built for eager emission");
    if (x0 == 0 && n_px == net.in_w) return idf_push_segment(s, stream_ids, n_ids, dev_pixels, 1);
    const bool first_mfma = !s->mfma.empty() && s->mfma[0] == 1;
    if (net.g[0].kind != IDF_CONV) return fail(IDF_EUNSUPPORTED, "pixel segments need a convolution as the first layer");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        if (s->h[id].x_next != x0)
            return fail(IDF_ESTATE, "stream %d: next column is %d, not %d", id, s->h[id].x_next, x0);
    }
    s->part.on = true; s->part.x_lo = x0; s->part.x_hi = x0 + n_px; s->part.first = x0 == 0; s->part.last = x0 + n_px == net.in_w;
    if (s->part.last) {
        // the row is whole: everything a pushed row does, with layer 0 taking only these columns
        rc = idf_push_segment(s, stream_ids, n_ids, dev_pixels, 1);
        s->part = idf_streams::Part{};
        return rc;
    }
    // layer 0 takes the columns into its rolling buffer; nothing can be final yet
    if (s->stg2d) {
        // the row that is begun needs a slot nobody reads any more
        bool room = true;
        for (const RowProg &q : s->prog) {
            const RowProg &p = s->prog_same ? s->prog_all : q;
            room = room && p.in[0] + 1 - first_needed(net.g[0], p.out[0]) <= s->units[0].ring_rows;
        }
        if (!room) rc = stg_drain(s);
        if (rc != IDF_OK) { s->part = idf_streams::Part{}; return rc; }
    }
    std::map<int64_t, std::vector<std::pair<int, int>>> groups;
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        if (net.in_h > 0 && s->h[id].r >= net.in_h) { s->part = idf_streams::Part{}; return fail(IDF_ESTATE, "stream %d: sample complete", id); }
        groups[first_mfma || s->use_gather ? s->h[id].sample * net.in_h + s->h[id].r : s->h[id].r].push_back({i, id});
    }
    for (auto &kv : groups) {
        const int64_t r = kv.first;
        rc = for_each_selection(kv.second, [&](const StreamSel &sel) {
            if (s->use_gather) {                  // rows of c are formed when the row is whole: the pixels wait in the layer's ring
                GatherHead h{};
                GatherStep a;
                gather_take(s, r, 1, x0, x0 + n_px, a);
                h.n = 1; h.n_layers = (int)net.g.size();
                h.stats = (unsigned long long *)(s->ws + s->stats_off);
                h.n_in = 1; h.seg_rows = 1; h.in_stride = n_px * net.in_c; h.in[0] = dev_pixels;
                const double bytes = (double)sel.n * n_px * net.in_c * ev_bytes(net.precision);
                hipError_t e = launch_conv_gather(net.precision, h, &a, sel, false, launch_ctx(s, kKindConvGather, bytes, 0));
                return e == hipSuccess ? (int)IDF_OK : dev_fail(e, "pixel segment launch");
            }
            if (!first_mfma) {
                // any other first convolution: the generic kernel with the segment's column range; every row the input
                // row touches goes back to the rolling buffer
                const Geom &g = net.g[0];
                ConvStep c{};
                c.g = g; c.layer = 0; c.y0 = r; c.cnt = 1;
                c.o_lo = rows_final(g, r); c.o_fin = c.o_lo;
                c.o_hi = std::max(rows_touched(g, r + 1), rows_final(g, r + 1));
                if (c.o_hi <= c.o_lo) return (int)IDF_OK;          // the row reaches no output row (stride and padding skip it)
                c.ring_rows = g.k_h;
                c.in = dev_pixels; c.in_stream_stride = (int64_t)n_px * net.in_c; c.in_row0 = r; c.in_by_position = 1;
                c.ring = s->ws + s->ring_off[0]; c.ring_stream_stride = s->ring_stride[0];
                c.dst = nullptr; c.dst_row0 = c.o_lo; c.out_cap = s->out_cap;
                c.w = s->ws + s->w_off[0];
                c.bias = net.b_img[0].empty() ? nullptr : s->ws + s->b_off[0];
                c.stats = (unsigned long long *)(s->ws + s->stats_off); c.n_layers = (int)net.g.size();
                c.x_lo = x0; c.x_hi = x0 + n_px; c.cont = x0 != 0;
                conv_generic_plan(c);
                hipError_t e = launch_conv_generic(net.precision, c, sel, launch_ctx(s, kKindConvGeneric, conv_step_bytes(net, c, sel.n), 0));
                return e == hipSuccess ? (int)IDF_OK : dev_fail(e, "pixel segment launch");
            }
            // the matrix-core kernel forms its rows of c when the row is whole: the pixels wait in the layer's ring
            RowBatch b;
            b.n = 1;
            take_step(s, 0, kv.first, 1, dev_pixels, 0, 1, kv.first, b.st[0]);
            return launch_rows(s, b, sel, (double)sel.n * n_px * net.in_c * ev_bytes(net.precision), 0);
        });
        if (rc != IDF_OK) break;
    }
    s->part = idf_streams::Part{};
    if (rc != IDF_OK) return rc;
    for (int i = 0; i < n_ids; ++i) s->h[stream_ids ? stream_ids[i] : i].x_next = x0 + n_px;
    return IDF_OK;
}

int idf_read_outputs(idf_streams *s, const int32_t *stream_ids, int n_ids, void *dev_out, int64_t max_rows,
                     int64_t *first_row, int32_t *n_rows)
{
    if (!s || !dev_out || !first_row || !n_rows) return fail(IDF_EINVAL, "null argument");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    if (max_rows < 1) return fail(IDF_EINVAL, "max_rows must be >= 1");
    if (s->eager.on) return fail(IDF_ESTATE, "eager emission: the output is read with idf_read_announced");
    if (s->since_read > 0) { s->read_each = s->since_read == 1; s->since_read = 0; }
    rc = pipeline_drain(s);                // rows still between stages belong to what was pushed
    if (rc != IDF_OK) return rc;
    rc = head_catch_up(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    const idf_net &net = *s->net;
    std::map<std::pair<int64_t, int>, std::vector<std::pair<int, int>>> groups;
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        const StreamHost &h = s->h[id];
        const int64_t n = std::min<int64_t>(h.out_written - h.out_read, max_rows);
        first_row[i] = net.out_h > 0 ? h.out_read % net.out_h : h.out_read;
        n_rows[i] = (int32_t)n;
        if (n > 0) groups[{h.out_read % s->out_cap, (int)n}].push_back({i, id});
    }
    CopyOut a{};
    a.src = s->ws + s->out_off; a.src_stream_stride = s->out_stride; a.out_cap = s->out_cap;
    a.dst = dev_out; a.row_elems = (int64_t)net.out_w * net.out_c; a.dst_stream_stride = max_rows * a.row_elems;
    a.elem_bytes = 4;
    for (auto &kv : groups) {
        const int64_t slot = kv.first.first;
        const int n = kv.first.second;
        rc = for_each_selection(kv.second, [&](const StreamSel &sel) {
            hipError_t e = launch_copy_out(a, sel, slot, n,
                                           launch_ctx(s, kKindCopyOut, 8.0 * n * a.row_elems * sel.n));
            return e == hipSuccess ? IDF_OK : dev_fail(e, "copy launch");
        });
        if (rc != IDF_OK) return rc;
    }
    for (int i = 0; i < n_ids; ++i) s->h[stream_ids ? stream_ids[i] : i].out_read += n_rows[i];
    return IDF_OK;
}

int idf_reset_streams(idf_streams *s, const int32_t *stream_ids, int n_ids)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    rc = pipeline_drain(s);
    if (rc != IDF_OK) return rc;
    const size_t per = s->net->g.size() * 2 * sizeof(unsigned long long);
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        hipError_t e = launch_fill_zero(s->ws + s->stats_off + per * id, per, s->st);
        if (e == hipSuccess) e = launch_fill_zero(s->ws + s->issued_off + per / 2 * id, per / 2, s->st);
        if (e == hipSuccess)
            e = launch_fill_zero(s->ws + s->head_off + (size_t)id * s->net->out_c * sizeof(double),
                                 (size_t)s->net->out_c * sizeof(double), s->st);
        if (e != hipSuccess) return dev_fail(e, "reset_streams");
        s->h[id] = StreamHost{};
        if (s->stg2d) { prog_split(s); s->prog[id] = RowProg{}; }
    }
    if (s->stg2d) prog_join(s);
    return IDF_OK;
}

int idf_get_stats(idf_streams *s, int stream_id, uint64_t *events_in, uint64_t *macs_executed, uint64_t *state_bytes)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    if (stream_id < 0 || stream_id >= s->B) return fail(IDF_EINVAL, "stream id %d outside [0, %d)", stream_id, s->B);
    const int n = (int)s->net->g.size();
    std::vector<unsigned long long> buf((size_t)n * 2);
    if (int rc = pipeline_drain(s)) return rc;
    if (int rc = count_waiting_rows(s)) return rc;
    hipError_t e = hipStreamSynchronize(s->st);
    if (e == hipSuccess)
        e = hipMemcpy(buf.data(), s->ws + s->stats_off + (size_t)stream_id * n * 2 * sizeof(unsigned long long),
                      buf.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return dev_fail(e, "get_stats");
    const int eb = ev_bytes(s->net->precision);
    for (int l = 0; l < n; ++l) {
        if (events_in) events_in[l] = buf[2 * l];
        if (macs_executed) macs_executed[l] = buf[2 * l + 1];
        if (state_bytes)
            state_bytes[l] = s->net->g[l].kind == IDF_CONV ? (uint64_t)s->ring_stride[l] * 4 : (uint64_t)s->held_stride[l] * eb;
    }
    return IDF_OK;
}

int idf_count_issued_macs(idf_streams *s, int on)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "eager emission keeps no count of issued multiply-adds");
    int rc = pipeline_drain(s);                 // what is on its way was pushed under the old setting
    if (rc != IDF_OK) return rc;
    s->count_issued = on != 0;
    return IDF_OK;
}

int idf_set_event_path(idf_streams *s, int events_per_kstep)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    if (events_per_kstep < 0) return fail(IDF_EINVAL, "events per K-step %d is negative", events_per_kstep);
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "eager emission has one kernel per layer kind and no event-list variant");
    int rc = pipeline_drain(s);                 // what is on its way was pushed under the old setting
    if (rc != IDF_OK) return rc;
    // (nets without a layer that could take it run as they do without it)
    bool any = false;
    for (const RowUnit &u : s->units) any = any || s->net->g[u.l].c_in <= kEventChannels;
    s->ev_per_step = any ? std::min(events_per_kstep, 1 << 16) : 0;
    return IDF_OK;
}

int idf_get_issued_macs(idf_streams *s, int stream_id, uint64_t *macs_issued)
{
    if (!s || !macs_issued) return fail(IDF_EINVAL, "null argument");
    if (stream_id < 0 || stream_id >= s->B) return fail(IDF_EINVAL, "stream id %d outside [0, %d)", stream_id, s->B);
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "eager emission keeps no count of issued multiply-adds");
    const int n = (int)s->net->g.size();
    std::vector<unsigned long long> iss((size_t)n), st((size_t)n * 2);
    if (int rc = pipeline_drain(s)) return rc;
    hipError_t e = hipStreamSynchronize(s->st);
    if (e == hipSuccess)
        e = hipMemcpy(iss.data(), s->ws + s->issued_off + (size_t)stream_id * n * sizeof(unsigned long long),
                      iss.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost);
    if (e == hipSuccess)
        e = hipMemcpy(st.data(), s->ws + s->stats_off + (size_t)stream_id * n * 2 * sizeof(unsigned long long),
                      st.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return dev_fail(e, "get_issued_macs");
    // the generic kernels test every value and keep no count of their own: they issue what they execute
    const bool own_count = s->use_gather || !s->mfma.empty();
    for (int l = 0; l < n; ++l) {
        const bool counted = s->use_gather || (own_count && l < (int)s->mfma.size() && s->mfma[l] == 1);
        macs_issued[l] = counted ? iss[l] : st[2 * l + 1];
    }
    return IDF_OK;
}

int idf_set_push_batching(idf_streams *s, int k)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    if (k < 1 || k > kGatherSegs) return fail(IDF_EINVAL, "pushes per launch %d outside [1, %d]", k, kGatherSegs);
    if (!s->use_cascade1d) return fail(IDF_EUNSUPPORTED, "holding back pushes is built for nets served by the 1-D cascade");
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "eager emission delivers every segment at once");
    int rc = pipeline_drain(s);                  // what is held back was pushed under the old setting
    if (rc != IDF_OK) return rc;
    rc = gather_rings(s, k);
    if (rc != IDF_OK) return rc;
    s->batch = k;
    return IDF_OK;
}

int idf_rows_pushed(const idf_streams *s, int stream_id, int64_t *rows)
{
    if (!s || !rows) return fail(IDF_EINVAL, "null argument");
    if (stream_id < 0 || stream_id >= s->B) return fail(IDF_EINVAL, "stream id %d outside [0, %d)", stream_id, s->B);
    *rows = s->h[stream_id].r;
    return IDF_OK;
}

int idf_snapshot_bytes(const idf_streams *s, size_t *bytes)
{
    if (!s || !bytes) return fail(IDF_EINVAL, "null argument");
    size_t total = 0;
    for_each_state_piece(s, 0, 0, [&](size_t, size_t n) { total += align_up(n, 16); });
    *bytes = total;
    return IDF_OK;
}

int idf_snapshot(idf_streams *s, int stream_id, void *dev_buf, idf_stream_pos *pos)
{
    if (!s || !dev_buf || !pos) return fail(IDF_EINVAL, "null argument");
    if (stream_id < 0 || stream_id >= s->B) return fail(IDF_EINVAL, "stream id %d outside [0, %d)", stream_id, s->B);
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "snapshots do not cover the maps of eager emission");
    if (s->head_units) return fail(IDF_EUNSUPPORTED, "snapshots do not cover the fully connected output units");
    if (s->h[stream_id].x_next != 0) return fail(IDF_ESTATE, "stream %d: a row is half presented", stream_id);
    int rc = pipeline_drain(s);
    if (rc != IDF_OK) return rc;
    rc = count_waiting_rows(s);
    if (rc != IDF_OK) return rc;
    const int32_t id32 = stream_id;
    rc = head_catch_up(s, &id32, 1);
    if (rc != IDF_OK) return rc;
    const StreamHost &h = s->h[stream_id];
    if (h.out_written != h.out_read) return fail(IDF_ESTATE, "stream %d: %lld completed output rows not read yet", stream_id,
                                                 (long long)(h.out_written - h.out_read));
    size_t at = 0;
    hipError_t e = hipSuccess;
    for_each_state_piece(s, stream_id, h.sample * s->net->in_h + h.r, [&](size_t off, size_t n) {
        if (e == hipSuccess && n) e = hipMemcpyAsync((char *)dev_buf + at, s->ws + off, n, hipMemcpyDeviceToDevice, s->st);
        at += align_up(n, 16);
    });
    if (e != hipSuccess) return dev_fail(e, "snapshot");
    pos->rows_pushed = h.r; pos->out_rows = h.out_written; pos->head_rows = h.head_done - h.head_base;
    return IDF_OK;
}

int idf_restore(idf_streams *s, int stream_id, const void *dev_buf, const idf_stream_pos *pos)
{
    if (!s || !dev_buf || !pos) return fail(IDF_EINVAL, "null argument");
    if (stream_id < 0 || stream_id >= s->B) return fail(IDF_EINVAL, "stream id %d outside [0, %d)", stream_id, s->B);
    const idf_net &net = *s->net;
    if (pos->rows_pushed < 0 || (net.in_h > 0 && pos->rows_pushed >= net.in_h) || pos->out_rows < 0 ||
        pos->head_rows < 0 || pos->head_rows > pos->out_rows)
        return fail(IDF_EINVAL, "inconsistent stream position");
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "snapshots do not cover the maps of eager emission");
    if (s->head_units) return fail(IDF_EUNSUPPORTED, "snapshots do not cover the fully connected output units");
    int rc = pipeline_drain(s);
    if (rc != IDF_OK) return rc;
    StreamHost &h = s->h[stream_id];
    if (h.out_written != h.out_read) return fail(IDF_ESTATE, "stream %d: %lld completed output rows not read yet", stream_id,
                                                 (long long)(h.out_written - h.out_read));
    size_t at = 0;
    hipError_t e = hipSuccess;
    for_each_state_piece(s, stream_id, (net.out_h > 0 ? pos->out_rows / net.out_h : 0) * net.in_h + pos->rows_pushed, [&](size_t off, size_t n) {
        if (e == hipSuccess && n) e = hipMemcpyAsync(s->ws + off, (const char *)dev_buf + at, n, hipMemcpyDeviceToDevice, s->st);
        at += align_up(n, 16);
    });
    if (e != hipSuccess) return dev_fail(e, "restore");
    h.r = pos->rows_pushed; h.out_written = h.out_read = pos->out_rows; h.x_next = 0;
    h.head_done = pos->out_rows; h.head_base = pos->out_rows - pos->head_rows;
    // the ring slots of the rows that came back follow from how many rows the stream has received; what waits in
    // front of a pool was counted when the snapshot was taken
    h.sample = net.out_h > 0 ? pos->out_rows / net.out_h : 0;
    h.early = early_at(s, h.r);
    if (s->stg2d) { prog_split(s); s->prog[stream_id] = prog_at(s, h.sample * net.in_h + h.r, true); prog_join(s); }
    return IDF_OK;
}

int idf_query_eager_bytes(const idf_net *net, int n_streams, int max_seg_rows, size_t *bytes)
{
    if (!net || !bytes || n_streams < 1 || max_seg_rows < 1) return fail(IDF_EINVAL, "bad argument");
    if (net->in_h <= 0) return fail(IDF_EUNSUPPORTED, "eager emission keeps the output map whole: the sample height must be known");
    *bytes = eager_layout(*net, n_streams, max_seg_rows, nullptr);
    return IDF_OK;
}

int idf_enable_eager(idf_streams *s, void *dev_workspace, size_t workspace_bytes)
{
    if (!s || !dev_workspace) return fail(IDF_EINVAL, "null argument");
    size_t need = 0;
    int rc = idf_query_eager_bytes(s->net, s->B, s->max_seg, &need);
    if (rc != IDF_OK) return rc;
    if (workspace_bytes < need) return fail(IDF_EINVAL, "eager workspace of %zu bytes, %zu needed", workspace_bytes, need);
    if (s->head_on) return fail(IDF_EUNSUPPORTED, "the averaging units read completed rows, eager emission has none");
    for (const StreamHost &h : s->h)
        if (h.r != 0 || h.out_written != 0 || h.x_next != 0) return fail(IDF_ESTATE, "eager emission must be enabled before the first push");
    eager_layout(*s->net, s->B, s->max_seg, &s->eager);
    s->eager.ws = (char *)dev_workspace;
    std::vector<double> macs;
    s->eager.one_launch = eager_one_launch(s, macs, s->eager.by_stage);
    if (s->eager.one_launch) eager_stages(s, macs);
    if (s->eager.by_stage && s->eager.parts == 0) s->eager.one_launch = s->eager.by_stage = false;
    s->eager.recorded = eager_recording(s) != 0;
    if (s->eager.stages > 1 && !s->eager.recorded) {
        hipError_t e = launch_fill(s->eager.open, 4, 1u, s->st);
        if (e != hipSuccess) return dev_fail(e, "enable_eager");
    }
    s->eager.on = true;
    return IDF_OK;
}

int idf_eager_state_bytes(const idf_streams *s, size_t *per_stream, int *rows_kept)
{
    if (!s || !per_stream) return fail(IDF_EINVAL, "null argument");
    if (!s->eager.on) return fail(IDF_ESTATE, "eager emission is not enabled");
    const idf_streams::Eager &E = s->eager;
    const int n = (int)s->net->g.size();
    size_t total = 0;
    for (int lv = 0; lv <= n; ++lv) {
        const bool has_c = lv > 0 && s->net->g[lv - 1].kind == IDF_CONV;
        // state c and the announced values; the deltas live only during a push, the last level's announced map is the output
        total += (size_t)E.row_elems[lv] * 4 * ((has_c ? E.cd_rows[lv] : 0) + (lv < n ? E.ann_rows[lv] : 0));
        if (rows_kept) rows_kept[lv] = E.cd_rows[lv];
    }
    *per_stream = total;
    return IDF_OK;
}

int idf_read_announced(idf_streams *s, int level, const int32_t *stream_ids, int n_ids, void *dev_out)
{
    if (!s || !dev_out) return fail(IDF_EINVAL, "null argument");
    if (!s->eager.on) return fail(IDF_ESTATE, "eager emission is not enabled");
    const int n = (int)s->net->g.size();
    if (level < 0 || level > n) return fail(IDF_EINVAL, "level %d outside [0, %d]", level, n);
    if (s->eager.ring && level != n)
        return fail(IDF_ESTATE, "level %d keeps a ring of %d rows, not its whole map: read them with idf_read_announced_rows", level,
                    s->eager.ann_rows[level]);
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    rc = eager_settle(s);
    if (rc != IDF_OK) return rc;
    const size_t bytes = (size_t)s->eager.rows[level] * s->eager.row_elems[level] * 4;
    // streams lie side by side, as they do in the output: one copy per run of ids
    for (int i = 0, run; i < n_ids; i += run) {
        const int id = stream_ids ? stream_ids[i] : i;
        for (run = 1; i + run < n_ids && (stream_ids ? stream_ids[i + run] : i + run) == id + run; ++run) {}
        hipError_t e = hipMemcpyAsync((char *)dev_out + (size_t)i * bytes, s->eager.ws + s->eager.ann_off[level] + (size_t)id * bytes,
                                      bytes * run, hipMemcpyDeviceToDevice, s->st);
        if (e != hipSuccess) return dev_fail(e, "read_announced");
    }
    return IDF_OK;
}

int idf_read_announced_rows(idf_streams *s, int level, const int32_t *stream_ids, int n_ids, void *dev_out, int max_rows,
                            int64_t *first_row, int32_t *n_rows)
{
    if (!s || !dev_out || !first_row || !n_rows) return fail(IDF_EINVAL, "null argument");
    if (!s->eager.on) return fail(IDF_ESTATE, "eager emission is not enabled");
    const idf_streams::Eager &E = s->eager;
    const int n = (int)s->net->g.size();
    if (level < 0 || level > n) return fail(IDF_EINVAL, "level %d outside [0, %d]", level, n);
    if (max_rows < 1) return fail(IDF_EINVAL, "max_rows must be >= 1");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    rc = eager_settle(s);
    if (rc != IDF_OK) return rc;
    const size_t row_bytes = (size_t)E.row_elems[level] * 4;
    std::vector<int64_t> lo, hi;
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        // rows of the level reached by the input rows seen so far; the newest `rows kept` of them are still there
        eager_bands(*s->net, 0, s->h[id].eager_rows, false, lo, hi);
        const bool whole = !E.ring || level == n;             // kept whole and cleared when the sample began
        const int64_t reached = whole ? (s->h[id].eager_rows > 0 ? E.rows[level] : 0) : hi[level];
        const int64_t first = whole ? 0 : std::max<int64_t>(0, reached - E.ann_rows[level]);
        const int64_t cnt = std::min<int64_t>(reached - first, max_rows);
        first_row[i] = first; n_rows[i] = (int32_t)cnt;
        if (E.one_launch && level > 0 && level < n && s->net->g[level - 1].kind == IDF_CONV) {      // not kept: f of the state
            hipError_t e = launch_eager_announced(s->net->precision, s->net->g[level - 1], s->eager.ws + E.c_off[level] + (size_t)id * E.cd_rows[level] * row_bytes,
                                                  E.cd_rows[level], first, (int)cnt, (char *)dev_out + (size_t)i * max_rows * row_bytes, s->st);
            if (e != hipSuccess) return dev_fail(e, "read_announced_rows");
            continue;
        }
        const char *src = s->eager.ws + E.ann_off[level] + (size_t)id * E.ann_rows[level] * row_bytes;
        for (int64_t r = first; r < first + cnt; ++r) {         // (a ring wraps: row by row)
            hipError_t e = hipMemcpyAsync((char *)dev_out + ((size_t)i * max_rows + (size_t)(r - first)) * row_bytes,
                                          src + (size_t)(r % E.ann_rows[level]) * row_bytes, row_bytes, hipMemcpyDeviceToDevice, s->st);
            if (e != hipSuccess) return dev_fail(e, "read_announced_rows");
        }
    }
    return IDF_OK;
}

int idf_enable_head(idf_streams *s)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    if (s->eager.on) return fail(IDF_EUNSUPPORTED, "the averaging units read completed rows, eager emission has none");
    for (const StreamHost &h : s->h)
        if (h.r != 0 || h.out_written != 0) return fail(IDF_ESTATE, "the averaging units must be enabled before the first push");
    s->head_on = true;
    return IDF_OK;
}

int idf_query_head_units_bytes(const idf_net *net, int n_streams, int n_units, size_t *bytes)
{
    if (!net || !bytes || n_streams < 1 || n_units < 1) return fail(IDF_EINVAL, "bad argument");
    if (net->out_h <= 0) return fail(IDF_EUNSUPPORTED, "output units have one weight per position: the sample height must be known");
    const size_t map = (size_t)net->out_h * net->out_w * net->out_c;
    *bytes = align_up(((size_t)n_units * map + n_units) * 4) + align_up((size_t)n_streams * n_units * sizeof(double));
    return IDF_OK;
}

int idf_enable_head_units(idf_streams *s, int n_units, const float *weights, const float *bias, void *dev_buf, size_t bytes)
{
    if (!s || !weights || !dev_buf) return fail(IDF_EINVAL, "null argument");
    size_t need = 0;
    int rc = idf_query_head_units_bytes(s->net, s->B, n_units, &need);
    if (rc != IDF_OK) return rc;
    if (bytes < need) return fail(IDF_EINVAL, "buffer of %zu bytes for the output units, %zu needed", bytes, need);
    rc = idf_enable_head(s);                       // the units ride on the averaging units' bookkeeping
    if (rc != IDF_OK) return rc;
    const size_t map = (size_t)s->net->out_h * s->net->out_w * s->net->out_c;
    hipError_t e = launch_fill_zero(dev_buf, need, s->st);
    if (e == hipSuccess) e = hipMemcpyAsync(dev_buf, weights, (size_t)n_units * map * 4, hipMemcpyHostToDevice, s->st);
    if (e == hipSuccess && bias)
        e = hipMemcpyAsync((char *)dev_buf + (size_t)n_units * map * 4, bias, (size_t)n_units * 4, hipMemcpyHostToDevice, s->st);
    if (e == hipSuccess) e = hipStreamSynchronize(s->st);          // the host arrays may go after the call
    if (e != hipSuccess) return dev_fail(e, "enable_head_units");
    s->head_units = n_units; s->head_units_ws = (char *)dev_buf; s->head_units_bias = bias != nullptr;
    return IDF_OK;
}

int idf_read_head_units(idf_streams *s, const int32_t *stream_ids, int n_ids, double *values, int64_t *rows)
{
    if (!s || !values || !rows) return fail(IDF_EINVAL, "null argument");
    if (!s->head_units) return fail(IDF_ESTATE, "no output units enabled");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    rc = pipeline_drain(s);
    if (rc != IDF_OK) return rc;
    rc = head_catch_up(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    const int k = s->head_units;
    const size_t map = (size_t)s->net->out_h * s->net->out_w * s->net->out_c;
    std::vector<double> all((size_t)s->B * k);
    std::vector<float> b(k, 0.f);
    hipError_t e = hipStreamSynchronize(s->st);
    if (e == hipSuccess)
        e = hipMemcpy(all.data(), s->head_units_ws + align_up(((size_t)k * map + k) * 4), all.size() * sizeof(double), hipMemcpyDeviceToHost);
    if (e == hipSuccess && s->head_units_bias)
        e = hipMemcpy(b.data(), s->head_units_ws + (size_t)k * map * 4, (size_t)k * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return dev_fail(e, "read_head_units");
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        rows[i] = s->h[id].head_done - s->h[id].head_base;
        // a unit that has received no row yet still states its bias (a constant input, Sec. 3)
        for (int u = 0; u < k; ++u) values[(size_t)i * k + u] = rows[i] > 0 ? all[(size_t)id * k + u] : (double)b[u];
    }
    return IDF_OK;
}

int idf_read_head(idf_streams *s, const int32_t *stream_ids, int n_ids, double *mean, int64_t *rows)
{
    if (!s || !mean || !rows) return fail(IDF_EINVAL, "null argument");
    if (!s->head_on) return fail(IDF_ESTATE, "the averaging units are not enabled");
    int rc = check_ids(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    rc = pipeline_drain(s);
    if (rc != IDF_OK) return rc;
    rc = head_catch_up(s, stream_ids, n_ids);
    if (rc != IDF_OK) return rc;
    const int c = s->net->out_c;
    std::vector<double> all((size_t)s->B * c);
    hipError_t e = hipStreamSynchronize(s->st);
    if (e == hipSuccess)
        e = hipMemcpy(all.data(), s->ws + s->head_off + (size_t)s->B * c * sizeof(double), all.size() * sizeof(double),
                      hipMemcpyDeviceToHost);
    if (e != hipSuccess) return dev_fail(e, "read_head");
    for (int i = 0; i < n_ids; ++i) {
        const int id = stream_ids ? stream_ids[i] : i;
        rows[i] = s->h[id].head_done - s->h[id].head_base;
        for (int k = 0; k < c; ++k) mean[(size_t)i * c + k] = rows[i] > 0 ? all[(size_t)id * c + k] : 0.0;
    }
    return IDF_OK;
}

int idf_measure_peak(int kind, void *dev_buf, size_t bytes, void *hip_stream, double *rate)
{
    if (!dev_buf || !rate) return fail(IDF_EINVAL, "null argument");
    if (kind < IDF_PEAK_COPY || kind > IDF_PEAK_MFMA_I8) return fail(IDF_EINVAL, "unknown kind %d", kind);
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess || cus < 1) return dev_fail(e, "measure_peak: device query");
    const bool copy = kind == IDF_PEAK_COPY;
    const int blocks = copy ? cus * 8 : cus * 2;             // two workgroups of four waves per compute unit: two waves per SIMD
    const int iters = 2048;
    if (bytes < ((size_t)1 << 20) || bytes < peak_sink_bytes(blocks))
        return fail(IDF_EINVAL, "measure_peak: the buffer holds %zu bytes, at least %zu are needed", bytes,
                    std::max<size_t>((size_t)1 << 20, peak_sink_bytes(blocks)));
    hipStream_t st = (hipStream_t)hip_stream;
    LaunchCtx lc;
    lc.st = st;
    e = launch_peak(kind, dev_buf, bytes, blocks, iters, lc);     // untimed: code and clocks warm
    hipEvent_t a = nullptr, b = nullptr;
    if (e == hipSuccess) e = hipEventCreate(&a);
    if (e == hipSuccess) e = hipEventCreate(&b);
    float best = 0.f;
    for (int rep = 0; rep < 3 && e == hipSuccess; ++rep) {
        lc.start = a; lc.stop = b;
        e = launch_peak(kind, dev_buf, bytes, blocks, iters, lc);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
        if (e == hipSuccess && (best == 0.f || ms < best)) best = ms;
    }
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
    if (e != hipSuccess) return dev_fail(e, "measure_peak");
    if (best <= 0.f) return fail(IDF_EDEVICE, "measure_peak: no time was measured");
    const double work = copy ? 2.0 * (double)(bytes / 32 * 16) : peak_ops(kind, blocks, iters);
    *rate = work / ((double)best * 1e-3) / (copy ? 1e9 : 1e12);
    return IDF_OK;
}

int idf_profile_begin(idf_streams *s)
{
    if (!s) return fail(IDF_EINVAL, "null argument");
    if (s->prof_on) return fail(IDF_ESTATE, "profiling already on");
    if (int rc = eager_flush(s)) return rc;
    s->prof_on = true;
    return IDF_OK;
}

int idf_profile_end(idf_streams *s, int max_kinds, idf_kernel_profile *out, int *n_kinds)
{
    if (!s || !out || !n_kinds || max_kinds < 1) return fail(IDF_EINVAL, "null argument");
    if (!s->prof_on) return fail(IDF_ESTATE, "profiling is not on");
    if (int rc = pipeline_drain(s)) return rc;
    s->prof_on = false;
    hipError_t e = hipStreamSynchronize(s->st);
    if (e != hipSuccess) return dev_fail(e, "profile_end");
    struct Agg { double ms = 0, bytes = 0; uint64_t cnt = 0; };
    std::map<std::pair<int, int>, Agg> agg;
    for (ProfRec &r : s->prof) {
        float t = 0.f;
        if (hipEventElapsedTime(&t, r.a, r.b) == hipSuccess) {
            Agg &g = agg[{r.kind, r.layer}];
            g.ms += t; g.bytes += r.bytes; g.cnt++;
        }
        s->ev_pool.push_back(r.a); s->ev_pool.push_back(r.b);
    }
    s->prof.clear();
    int n = 0;
    for (auto &kv : agg) {
        if (n >= max_kinds) break;
        memset(&out[n], 0, sizeof(out[n]));
        if (kv.first.second >= 0) snprintf(out[n].name, sizeof(out[n].name), "%s@%d", kind_name(kv.first.first), kv.first.second);
        else snprintf(out[n].name, sizeof(out[n].name), "%s", kind_name(kv.first.first));
        out[n].launches = kv.second.cnt; out[n].total_ms = kv.second.ms; out[n].algorithmic_bytes = kv.second.bytes;
        ++n;
    }
    *n_kinds = n;
    return IDF_OK;
}

const char *idf_layer_kernel(const idf_streams *s, int layer)
{
    if (!s || layer < 0 || layer >= (int)s->net->g.size()) return nullptr;
    if (s->use_gather) return kind_name(s->use_cascade1d ? kKindCascade1d : kKindConvGather);
    if (s->mfma[layer]) return kind_name(kKindConvMfma);
    return s->net->g[layer].kind == IDF_CONV ? kind_name(kKindConvGeneric) : kind_name(kKindPoolGeneric);
}

}  // extern "C"
