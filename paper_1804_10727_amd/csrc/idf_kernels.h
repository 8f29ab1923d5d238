// Launchers of the device kernels (defined in the k_*.hip files), called by the host side.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <type_traits>

#include "idf_common.h"

namespace idf {

// Where and how a kernel is launched: plain, or bracketed by an event pair stamped at the
// kernel's own start and end (profiling).
struct LaunchCtx {
    hipStream_t st = nullptr;
    hipEvent_t start = nullptr, stop = nullptr;
};

// (arguments by reference: by value a block of 3 KB was copied three times on its way, 0.03 to 0.11 us)
template <class... P>
inline hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, const LaunchCtx &c, const std::common_type_t<P> &...args)
{
    void *list[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    const void *fn = reinterpret_cast<const void *>(kernel);
    const hipError_t e = c.start ? hipExtLaunchKernel(fn, grid, block, list, lds, c.st, c.start, c.stop, 0) : hipLaunchKernel(fn, grid, block, list, lds, c.st);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

// A kernel as a type, and the one call that lets its launches have so much LDS: kernels of the same arguments have pointers of one
// type, so that a flag kept per type would be set for the first of them only.
template <auto K> struct Kernel { static constexpr auto entry = K; };
template <int BYTES, auto K> inline hipError_t allow_lds(Kernel<K>)
{
    static const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(K), hipFuncAttributeMaxDynamicSharedMemorySize, BYTES);
    return e;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits until every global
// store and atomic of the wave has been acknowledged (a release fence over all address spaces),
// a memory round trip that the kernels here do not need at their internal barriers: what the
// waves of a workgroup exchange goes through LDS.
__device__ __forceinline__ void lds_barrier()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier\n\ts_waitcnt lgkmcnt(0)" ::: "memory");
#endif
}

enum KernelKind { kKindConvGeneric = 0, kKindPoolGeneric, kKindCopyOut, kKindCascade1d, kKindConvMfma, kKindHead, kKindEager, kKindConvGather, kKindCount };
inline const char *kind_name(int k)
{
    static const char *names[kKindCount] = {"conv_generic", "pool_generic", "copy_out", "cascade1d", "conv3x3_mfma", "head_accumulate", "eager", "conv_gather"};
    return k >= 0 && k < kKindCount ? names[k] : "?";
}

// Generic kernels: any layer shape, any precision (prec = IDF_PREC_*).
hipError_t launch_conv_generic(int prec, const ConvStep &a, const StreamSel &sel, const LaunchCtx &lc);
hipError_t launch_pool_generic(int prec, const PoolStep &a, const StreamSel &sel, const LaunchCtx &lc);
hipError_t launch_head_units(const HeadUnits &a, const StreamSel &sel, int64_t first_slot, int n_rows, const LaunchCtx &lc);
hipError_t launch_head_accumulate(const HeadAcc &a, const StreamSel &sel, int64_t first_slot, int n_rows, const LaunchCtx &lc);
// what: 0 = pushed rows become the announced input, 1 = conv layer, 2 = pool layer
hipError_t launch_eager(int prec, int what, const EagerStep &a, const StreamSel &sel, const LaunchCtx &lc);
// A segment through a whole net of 3x3 conv layers and 2x2 pools in one launch: fills in how its bands lie (false: they
// are too large for it), and the launch.
bool eager_pass_shape(int prec, EagerPass &a);
hipError_t launch_eager_pass(int prec, const EagerPass &a, int stages, bool small, const StreamSel &sel, const LaunchCtx &lc);
// Announced values of rows [first, first + n) of a conv layer from its ring of c_rows rows of state.
hipError_t launch_eager_announced(int prec, const Geom &g, const void *c, int c_rows, int64_t first, int n, void *out, hipStream_t st);
// Sets the 4-byte words of bytes (a multiple of 4, 4-byte aligned) with a kernel on stream st.
hipError_t launch_fill(void *p, size_t bytes, uint32_t v, hipStream_t st);
inline hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t st) { return launch_fill(p, bytes, 0u, st); }
hipError_t launch_copy_out(const CopyOut &a, const StreamSel &sel, int64_t first_slot, int n_rows,
                           const LaunchCtx &lc);

// Does the gathering kernel take the whole of this 1-D net?
bool cascade1d_eligible(int prec, const Geom *g, int n_layers, int max_seg_rows);

// Matrix-core kernel for 3x3 / stride 1 / same-padded conv layers.
int conv3x3_mfma_vl(int prec);
bool conv3x3_mfma_eligible(int prec, const Geom &g);
// Packs weights [k_h][k_w][c_in][c_out] into fragment order; returns the size (out may be null).
size_t conv3x3_mfma_pack(int prec, const Geom &g, const void *w_khkwcico, void *out);
// Where in that packing the event-path weights of an int8 layer begin (0: the layer has none), and the
// most events per 32 positions of a row's stretch the event path takes.
size_t conv3x3_mfma_event_weights(int prec, const Geom &g);
int conv3x3_mfma_event_cap();
// Fills in how the workgroups of a step of a.n_rows rows lie (a.n_rows and a.ev_limit are set).  narrow: the step may share a
// launch with one that takes the event path.  launch_waves: conv3x3_mfma_wide_waves of all steps of the launch, which count from kWideLaunch on.
constexpr int kWideLaunch = 1400;
int64_t conv3x3_mfma_wide_waves(int prec, const Geom &g, int n_streams, const RowStep &a);
void conv3x3_mfma_shape(int prec, const Geom &g, int n_streams, bool narrow, int64_t launch_waves, RowStep &a);
// Tiles per stream and step that a launch takes; a step of more is cut after as many rows as fit (false: not even two do).
constexpr int kRowTilesMax = 65535;
bool conv3x3_mfma_split(RowStep &first, RowStep &rest);
hipError_t launch_conv3x3_mfma_rows(int prec, const RowBatch &b, const StreamSel &sel, const LaunchCtx &lc);

// Matrix-core kernel that gathers its windows from memory: any kernel size, strides 1, 2, 4 .., any padding.
void conv_gather_layer(int prec, const Geom &g, GatherStep &a);
bool conv_gather_takes(int prec, const Geom &g, int ring_rows);
double conv_gather_traffic(int prec, const Geom &g, int n_streams, int rows);
void conv_gather_shape(bool first, GatherStep &a);
size_t conv_gather_pack(int prec, const Geom &g, const void *w_khkwcico, void *out);
// chain: the steps one after the other (a workgroup per stream), else all side by side.
hipError_t launch_conv_gather(int prec, const GatherHead &h, const GatherStep *st, const StreamSel &sel, bool chain, const LaunchCtx &lc);

hipError_t launch_ring_move(const RingMove &a, const LaunchCtx &lc);

// Plain kernels that show what the machine delivers (copy, multiply-add chains, matrix-instruction
// chains): bytes the compute kinds write for a launch of `blocks` workgroups, operations such a
// launch performs, and the launch itself (copy: first half of buf to the second half).
size_t peak_sink_bytes(int blocks);
double peak_ops(int kind, int blocks, int iters);
hipError_t launch_peak(int kind, void *buf, size_t bytes, int blocks, int iters, const LaunchCtx &lc);

// Largest number of touched output rows one generic conv step can take for a layer with
// c_out output channels (the host splits longer steps).
int conv_generic_max_rows(int c_out);
// Chooses tile_x / tile_c / cells_per_thread of a generic conv step.
void conv_generic_plan(ConvStep &a);

}  // namespace idf
