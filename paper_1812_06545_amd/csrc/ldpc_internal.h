// Internal declarations shared by the libldpc translation units.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <new>
#include <stdexcept>
#include <system_error>
#include <vector>

#include "ldpc.h"

#define LDPC_HIP_OR_RETURN(expr)                 \
    do {                                         \
        hipError_t ldpc_e_ = (expr);             \
        if (ldpc_e_ != hipSuccess)               \
            return LDPC_EDEVICE;                 \
    } while (0)

namespace ldpc {

// No C++ exception crosses the C interface: every entry point is a
// function-try-block whose handler calls this (inside the handler, so the
// exception in flight is rethrown and classified).  Host allocation and
// thread-creation failures become LDPC_ENOMEM; nothing else is expected to
// throw, and anything that does is reported as LDPC_EDEVICE.
inline ldpc_status status_of_exception() noexcept
{
    try {
        throw;
    } catch (const std::bad_alloc &) {
        return LDPC_ENOMEM;
    } catch (const std::length_error &) {
        return LDPC_ENOMEM;
    } catch (const std::system_error &) {
        return LDPC_ENOMEM;
    } catch (...) {
        return LDPC_EDEVICE;
    }
}

}  // namespace ldpc

namespace ldpc {

// Word of a frame's LDS where its messages start, after n posteriors and the
// dummies' constants (a multiple of 4).
#ifdef __HIPCC__
__host__ __device__
#endif
inline int32_t fused_first_message(int32_t n)
{
    return (n + 3 + 3) / 4 * 4;
}

// Address tables of the frame-resident kernel, in device memory.  Addresses
// are byte addresses of 4-byte words in a frame's LDS (fused_kernels.h gives
// the words' places and the lanes' roles); a lane's slots 4i .. 4i + 3 form a
// quad (16 bytes), and quads are indexed in 16-byte units.
//   row order  rows by descending degree (stable); group g is rows 32g .. of it.
//   row_grp    per group: (longest half) << 16 | message slots before the
//              group; first quad row / 64.
//   row_tab    [first + slot quad][64 lanes] posterior addresses.
//   col_grp    per 64 columns: longest column; first quad row / 64.
//   col_tab    [first + slot quad][64 lanes] message addresses in the padded
//              slot order, in ascending row order of the column's edges.
//   *_x        the same for messages in CSR order, with row_pos giving the
//              messages' addresses beside row_tab's posteriors; every group has
//              four quads.  Built only for codes whose padded order does not
//              fit a workgroup's LDS in some type in which CSR order does.
//   lay_ptr    per layer: its first group; then the group count.
//   lay_grp    per group of up to 16 rows of a layer: (longest quarter) << 8 |
//              rows; first quad.
//   lay_tab    per group: [slot quad][4 parts][rows] posterior addresses, then
//              the same of the messages in CSR order.
struct FusedTables {
    int32_t row_groups = 0;
    int32_t slot_words = 0;  // message words of the padded slot order
    int32_t row_words = 0, col_words = 0, lay_words = 0;  // sizes of row_tab, col_tab, lay_tab
    const int32_t *row_grp = nullptr, *row_tab = nullptr, *col_grp = nullptr, *col_tab = nullptr;
    const int32_t *row_grp_x = nullptr, *row_tab_x = nullptr, *row_pos_x = nullptr, *col_tab_x = nullptr;
    const int32_t *lay_ptr = nullptr, *lay_grp = nullptr, *lay_tab = nullptr;
};

}  // namespace ldpc

// A code handle: H in device memory, in two layouts.
//   CSR/CSC (every code): edges numbered in CSR order (rows ascending,
//   columns ascending inside a row); col_edge lists each column's edges in
//   ascending row order.  Used by the per-iteration streaming kernels.
//   Address tables (FusedTables) for the frame-resident kernel.
struct ldpc_code_s {
    int device = 0;
    int32_t m = 0, n = 0;
    int64_t E = 0;
    int32_t max_row_deg = 0, max_col_deg = 0;
    int64_t column_reads = 0;  // sum over the edges of their column's degree
    void *d_mem = nullptr;
    const int32_t *row_ptr = nullptr;   // m + 1
    const int32_t *col_idx = nullptr;   // E
    const int32_t *col_ptr = nullptr;   // n + 1
    const int32_t *col_edge = nullptr;  // E
    // circulant-block structure (is_qc)
    bool is_qc = false;
    int32_t mb = 0, Z = 0, nblocks = 0;
    int32_t qc_words = 0;  // words of a table of the block structure: part of the frame-resident kernel's fit rule
    // Address tables of the frame-resident kernel (codes that can fit it).
    ldpc::FusedTables fused;
    // Layers of the layered schedule (host): maximal runs of consecutive rows,
    // in ascending order, in which no two rows share a variable.  Layer l is
    // rows [layer_ptr[l], layer_ptr[l+1]); layer_dmax[l] its largest degree.
    std::vector<int32_t> layer_ptr, layer_dmax;
    int32_t layer_rows = 0;  // of the largest layer
    // Hash of the code's shape (sizes, lifting size, row and column degree
    // histograms): the key of tuning choices, which depend on shape only.
    uint64_t shape_hash = 0;
};

namespace ldpc {

constexpr int kChunk = 64;  // frames per wavefront in the streaming layout

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int64_t frames_padded(int64_t frames) { return (frames + kChunk - 1) / kChunk * kChunk; }

bool code_on_current_device(const ldpc_code_s *c);

// Timing of one kernel launch when profiling is on (and the stream is not
// being captured): the scope hands out a start and a stop event that the
// launch carries itself (LDPC_LAUNCH, i.e. hipExtLaunchKernelGGL), so the
// runtime stamps the kernel's own start and end and no separate event
// packet sits between dependent launches; the scope files the pair on exit.
// Otherwise both events are null and LDPC_LAUNCH is a plain launch.
class ProfScope {
  public:
    // enabled = false: no timing for this launch, whatever the global setting.
    ProfScope(ldpc_kernel_kind kind, hipStream_t stream, bool enabled = true);
    ~ProfScope();
    ProfScope(const ProfScope &) = delete;
    ProfScope &operator=(const ProfScope &) = delete;
    hipEvent_t start() const { return start_; }
    hipEvent_t stop() const { return stop_; }

  private:
    int kind_ = -1;
    hipEvent_t start_ = nullptr, stop_ = nullptr;
};

#define LDPC_LAUNCH(ps, kernel, grid, block, shmem, stream, ...)                                                  \
    do {                                                                                                         \
        if ((ps).start())                                                                                        \
            hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, (ps).start(), (ps).stop(), 0u, __VA_ARGS__); \
        else                                                                                                     \
            hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);                                \
    } while (0)

// Copies bytes (a multiple of 16, both pointers 16-byte aligned) with the
// streaming copy kernel on `stream`; either side may be pinned host memory
// mapped for the device.
ldpc_status launch_copy16(void *dst, const void *src, size_t bytes, hipStream_t stream);
// The same copy on a grid of at most max_blocks workgroups of 256 threads,
// for copies that cross the host link while other kernels run.
ldpc_status launch_link_copy16(void *dst, const void *src, size_t bytes, int32_t max_blocks, hipStream_t stream);

// Workspace bytes of one fused launch of ldpc_decode_batch (its job table
// and work counter).  A batch of J jobs needs at most J such launches.
size_t fused_group_bytes();

// ldpc_decode's frames as one frame-resident launch, if the code fits that kernel
// and it is the faster route (frame_resident_faster): true, with the call's status
// in *rc (nothing is left to do), or false, and the streaming path takes the
// call.  ws: at least 4 bytes of device memory of the call's own.  (MI355X, FP32,
// 10 iterations, us per call, frames 1 / 256 / 1024, streaming and frame-resident:
// qc n = 648 88 / 119 / 186 and 31 / 35 / 96; qc n = 3840, one frame to a CU,
// 125 / 273 / 761 and 111 / 131 / 505; n = 1999 of degrees 2 to 29 107 / 200 /
// 487 and 58 / 67 / 224; layered qc n = 1944 446 / 533 / 734 and 157 / 170 /
// 468; FP64 n = 504 131 / 156 / 304 and 25 / 29 / 82.)
bool fused_decode(const ldpc_job &job, ldpc_dtype dt, void *ws, hipStream_t stream, ldpc_status *rc);

// Streaming (per-iteration) path.
size_t stream_workspace_bytes(const ldpc_code_s *c, ldpc_dtype dt, int32_t frames, int32_t max_iter);
// ms_scale / ms_offset: the min-sum magnitude correction (used with
// LDPC_MIN_SUM; natural-LLR units).
ldpc_status stream_decode(const ldpc_code_s *c, ldpc_dtype dt, int32_t frames, int32_t max_iter, uint32_t flags,
                          const void *llr, uint8_t *bits, int32_t *iters, void *posterior, void *ws,
                          hipStream_t stream, double ms_scale, double ms_offset);
// Flooding of a few frames with one launch per iteration (few.hip), on the
// streaming workspace.  few_frames_groups: the groups of frames it would run, or 0
// where the check and variable kernels are the faster form.
int32_t few_frames_groups(const ldpc_code_s *c, bool f64, int32_t frames);
template <class A>
ldpc_status decode_few(const ldpc_code_s *c, int32_t frames, int32_t max_iter, uint32_t flags,
                       const typename A::T *llr, uint8_t *bits, int32_t *iters, typename A::T *post,
                       typename A::T *R, typename A::T *Lch, int32_t *done, int32_t *unsat, hipStream_t s,
                       typename A::T scale, typename A::T offset);
// scale finite and > 0, offset finite and >= 0.
bool minsum_params_ok(double scale, double offset);

}  // namespace ldpc
