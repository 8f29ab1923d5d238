// Stands in for the HIP runtime so that the library's host side can be run, and watched, without a GPU: allocations are
// addresses nobody dereferences, copies and launches do nothing.  What a launch of the 3x3 kernel would read and write is
// followed row by row: every row it reads must lie where an earlier launch has put it, every row of every layer must be
// formed once and in order.
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <map>
#include <string>
#include <utility>
#include <vector>

#define __host__
#define __device__
#include "idf_common.h"

using namespace idf;

namespace {

struct Dim3 { uint32_t x, y, z; };
std::map<const void *, std::string> g_names;
std::map<const void *, long> g_dynamic_lds;           // what a kernel has been allowed
std::map<const void *, long> g_large;                  // launches with more than 64 KB of it
std::string g_error;
long g_launches = 0, g_fail_at = -1, g_lds_limit = 160 * 1024 - 256;
int g_last = 0;
struct Config { Dim3 grid, block; size_t lds; void *stream; } g_config;
std::vector<std::pair<std::string, long>> g_count;
unsigned long long g_recording = 0;
long g_max_lds = 0;                                    // dynamic LDS of any launch

struct Row { int layer, y; };
std::map<uintptr_t, Row> g_rows;                       // address of a row in a ring -> what lies there
std::map<std::pair<int, int>, int> g_next;             // (stream, layer) -> next output row

void error(const std::string &what) { if (g_error.empty()) g_error = what; }
std::string str(long v) { return std::to_string(v); }

void rows_launch(const RowBatch &b, const StreamSel &sel, const Dim3 &grid, size_t lds, int eb)
{
    if (b.n < 1 || b.n > kRowBatchMax || (int)grid.z != b.n || (int)grid.x != sel.n) return error("grid does not fit the steps");
    if (grid.y < 1 || grid.y > 65535) return error("grid of " + str(grid.y) + " tiles");
    if ((long)lds > g_lds_limit) return error("LDS of " + str(lds));
    std::vector<std::pair<uintptr_t, Row>> writes;
    std::map<uintptr_t, int> reads;
    for (int k = 0; k < b.n; ++k) {                        // rows that a layer of another kind has put into a ring: here they are counted
        const RowStep &a = b.st[k];
        for (int i = 0; a.form == kRowTake && !a.in_new && i < sel.n; ++i)
            for (int r = 0; r < a.n_rows; ++r)
                g_rows[(uintptr_t)a.in_ring + (uintptr_t)((a.in_stride * (int64_t)sel_stream(sel, i) + (int64_t)((a.slot0 + r) % a.ring_rows) * a.w * a.c_in) * eb)] =
                    Row{a.layer, a.y0 + r};
    }
    for (int k = 0; k < b.n; ++k) {
        const RowStep &a = b.st[k];
        if (a.tiles < 1 || a.tiles > (int)grid.y) error("tiles of a step exceed the grid");
        for (int i = 0; i < sel.n; ++i) {
            const int stream = sel_stream(sel, i);
            const size_t row_bytes = (size_t)a.w * a.c_in * eb;
            const uintptr_t ring = (uintptr_t)a.in_ring + (uintptr_t)((int64_t)stream * a.in_stride * eb);
            if ((int64_t)a.in_stride < (int64_t)a.ring_rows * a.w * a.c_in) error("ring stride of layer " + str(a.layer));
            if (a.form == kRowTake) {
                if (a.tiles != a.n_rows) error("rows taken");
                if (a.in_new && a.new_stride < (int64_t)a.n_rows * (a.x_hi - a.x_lo) * a.c_in) error("stride of the caller's rows");
                for (int r = 0; r < a.n_rows; ++r)
                    if (a.in_new && a.y0 + r >= a.y_save) writes.push_back({ring + (size_t)((a.slot0 + r) % a.ring_rows) * row_bytes, Row{a.layer, a.y0 + r}});
                continue;
            }
            for (int y = a.y0 - 1; y <= a.y0 + a.n_rows; ++y) {
                if (y < 0 || y >= a.h || y >= a.y_new) continue;
                if (a.slot0 + (y - a.y0 + 1) >= 2 * a.ring_rows) error("window of layer " + str(a.layer) + " laps its ring");
                const uintptr_t at = ring + (size_t)((a.slot0 + (y - a.y0 + 1)) % a.ring_rows) * row_bytes;
                auto it = g_rows.find(at);
                if (it == g_rows.end() || it->second.layer != a.layer || it->second.y != y)
                    error("layer " + str(a.layer) + " stream " + str(stream) + " does not find row " + str(y));
                reads[at] = 1;
            }
            if (!a.pool_emit) continue;                // formed once more only to be counted
            int &next = g_next[{stream, a.layer}];
            if (a.y0 != next) error("layer " + str(a.layer) + " forms row " + str(a.y0) + " instead of " + str(next));
            next = (a.y0 + a.n_rows) % a.h;
            if (a.pool && a.y0 % 2) error("pool of layer " + str(a.layer) + " starts with an odd row");
            if (a.to_output || a.next_layer < 0) continue;
            const int w = a.pool ? a.w / 2 : a.w, first = a.pool ? a.y0 / 2 : a.y0;
            int n = a.pool ? a.n_rows / 2 : a.n_rows;
            for (int j = 0; j < n; ++j)
                writes.push_back({(uintptr_t)a.dst + (uintptr_t)((a.dst_stride * stream + (int64_t)((a.dst_slot0 + j) % a.dst_rows) * w * a.c_out) * eb),
                                  Row{a.next_layer, first + j}});
        }
    }
    for (auto &w : writes) if (reads.count(w.first)) error("a row is overwritten by the launch that reads it");
    std::map<uintptr_t, int> once;
    for (auto &w : writes) {
        if (once[w.first]++) error("two rows of a launch go to one place");
        g_rows[w.first] = w.second;
    }
}

int launch(const void *fn, Dim3 grid, void **args, size_t lds)
{
    const long at = g_launches++;
    if (at == g_fail_at) return g_last = 98;           // (a launch failure)
    const std::string &name = g_names[fn];
    if (grid.x < 1 || grid.y < 1 || grid.z < 1 || grid.y > 65535 || grid.z > 65535) error("grid of " + name);
    g_max_lds = (long)lds > g_max_lds ? (long)lds : g_max_lds;
    if (lds > 64 * 1024) ++g_large[fn];
    if (lds > 64 * 1024 && (long)lds > g_dynamic_lds[fn]) error("LDS of " + str(lds) + " that was not asked for: " + name);
    bool found = false;
    for (auto &c : g_count) if (c.first == name) { ++c.second; found = true; }
    if (!found) g_count.push_back({name, 1});
    if (name.find("k_conv3x3_mfma_rows") != std::string::npos)
        rows_launch(*(const RowBatch *)args[0], *(const StreamSel *)args[1], grid, lds,
                    name.find("TraitsF32") != std::string::npos ? 4 : name.find("TraitsBf16") != std::string::npos ? 2 : 1);
    return 0;
}

}  // namespace

extern "C" {

// ---- for the tests ----
long host_launches(const char *part)
{
    long n = 0;
    for (auto &c : g_count) if (!part || c.first.find(part) != std::string::npos) n += c.second;
    return n;
}
void host_record(unsigned long long id) { g_recording = id; }      // (0: the stream is not being recorded)
long host_max_lds() { return g_max_lds; }
long host_large_kernels() { return (long)g_large.size(); }
const char *host_error() { return g_error.c_str(); }
void host_fail_in(long n) { g_fail_at = n < 0 ? -1 : g_launches + n; }
void host_begin() { g_rows.clear(); g_next.clear(); g_error.clear(); g_count.clear(); g_large.clear(); g_fail_at = -1; g_max_lds = 0; }

// ---- the runtime ----
void **__hipRegisterFatBinary(const void *) { static void *handle[1]; return handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { g_names[fn] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) { g_config = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void *fn, Dim3 grid, Dim3, void **args, size_t lds, void *) { return launch(fn, grid, args, lds); }
int hipExtLaunchKernel(const void *fn, Dim3 grid, Dim3, void **args, size_t lds, void *, void *, void *, int) { return launch(fn, grid, args, lds); }
int hipGetLastError() { const int e = g_last; g_last = 0; return e; }
const char *hipGetErrorString(int e) { return e == 98 ? "a launch failure" : "an error"; }
int hipFuncSetAttribute(const void *fn, int attribute, int value)
{
    if (attribute == 8) g_dynamic_lds[fn] = value;     // hipFuncAttributeMaxDynamicSharedMemorySize
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)(uintptr_t)0x200000000ull; return 0; }
int hipMemcpy(void *dst, const void *, size_t n, int kind) { if (kind == 2) memset(dst, 0, n); return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamGetCaptureInfo(void *, int *status, unsigned long long *id) { *status = g_recording != 0; if (id) *id = g_recording; return 0; }
int hipEventCreate(void **) { return 2; }
int hipEventDestroy(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0; return 0; }

}  // extern "C"
