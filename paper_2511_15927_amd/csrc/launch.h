// Host-callable launchers of the scan kernels (defined in scan_inst.hip, one object per (d_state, lanes-per-chain)).
#pragma once
#include "kernels.h"

#include <atomic>

namespace bm {
// A launch with more than 64 KB of dynamic LDS is refused until its kernel's limit has been raised, once per device.  The flag
// is published after the limit is up: a thread that finds it unset raises the limit itself (that is idempotent) instead of
// launching under one that another thread is still raising.  A failure is the caller's to report; the next call tries again.
class LdsLimit {
public:
    hipError_t raise(const void* kernel, size_t bytes)
    {
        int dev = -1;
        const bool known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices;
        if (known && raised_[dev].load(std::memory_order_acquire)) return hipSuccess;
        const hipError_t err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (err == hipSuccess && known) raised_[dev].store(true, std::memory_order_release);
        return err;
    }

private:
    static constexpr int kMaxDevices = 64;
    std::atomic<bool> raised_[kMaxDevices] = {};
};

// Compute units of the current device (256 when no device answers), asked once per device; defined in bimamba_api.hip
// and used by the host-side plan and by every launcher, so that all of them size a launch for the same chip.
int cu_count();

// Launchers that return an error have launched nothing, or nothing but what writes the call's workspace.
#define BM_DECLARE_SCAN(n, s)                                                                                      \
    hipError_t launch_scan_n##n##_s##s(int a_scalar_per_head, int io_bf16, const SweepArgs& sa, const CarryArgs& ca, \
                                       int batch, int short_call, hipStream_t st, hipEvent_t ev_start,             \
                                       hipEvent_t ev_stop);
BM_DECLARE_SCAN(4, 1)
BM_DECLARE_SCAN(8, 1)
BM_DECLARE_SCAN(16, 1)
BM_DECLARE_SCAN(16, 2)
BM_DECLARE_SCAN(16, 4)
BM_DECLARE_SCAN(32, 1)
BM_DECLARE_SCAN(32, 2)
BM_DECLARE_SCAN(32, 4)
BM_DECLARE_SCAN(64, 1)
BM_DECLARE_SCAN(64, 4)
BM_DECLARE_SCAN(128, 1)
BM_DECLARE_SCAN(128, 4)
#undef BM_DECLARE_SCAN

// The one-row-per-chain form of short calls (row_kernels.h): whether a call takes it, and its shape.
struct RowForm {
    int tw, nseg, seg_len;
};
struct RowArgs;
bool row_form(int batch, int seqlen, int d_inner, int d_state, bool halves, RowForm* f);   // halves: the directions write halves of their own
bool row_reach(int batch, int seqlen, int d_inner);   // whether a call is of a size that the row form takes for some state count and combine
bool stack_form(int batch, int seqlen, int d_inner, int d_state, RowForm* f);      // the same for a stack of layers (stack_kernels.h)
struct StackArgs;
// apart: no two steps have outputs, no two layers states or tails in the same memory
hipError_t launch_stack(int io_bf16, const StackArgs& a, int batch, bool apart, hipStream_t st);
int stack_side_by_side(const StackArgs& a, int batch);   // steps side by side of such a stack, 0: one after the other (stack_kernels.h)
hipError_t launch_row(int io_bf16, const RowArgs& a, int batch, hipStream_t st);   // (an error: nothing was launched)

struct SsdPrepPair;
struct SsdArgs;
struct SsdCarryArgs;
struct SsdStatePair;
bool ssd_supported(int d_state, int headdim);
hipError_t launch_ssd_prep(int d_state, const SsdPrepPair& pa, int nchunk, int batch, hipStream_t st);   // (an error: nothing was launched)
hipError_t launch_ssd_scan(int d_state, int headdim, const SsdStatePair& sp, int dirs, int batch, hipStream_t st);
// (defined in ssd_wide_inst.hip, one object per (d_state, head width))
hipError_t launch_ssd_wide_n128_p64(const SsdStatePair& sp, int dirs, int batch, hipStream_t st);
hipError_t launch_ssd_wide_n128_p32(const SsdStatePair& sp, int dirs, int batch, hipStream_t st);
hipError_t launch_ssd_wide_n64_p64(const SsdStatePair& sp, int dirs, int batch, hipStream_t st);
hipError_t launch_ssd_wide_n64_p32(const SsdStatePair& sp, int dirs, int batch, hipStream_t st);
void launch_ssd_carry(int d_state, const SsdCarryArgs& ca, hipStream_t st);
struct SsdBlockArgs;
hipError_t launch_ssd_block_prep(int d_state, const SsdBlockArgs& a, hipStream_t st);   // (calls of one chunk: ssd_block.h)
hipError_t launch_ssd_block(int d_state, const SsdBlockArgs& a, hipStream_t st);   // (an error: nothing was launched)
int ssd_block_tiles(int d_state, const SsdBlockArgs& a);   // SsdBlockArgs::tiles of a call that goes in one launch, else 0
void launch_ssd_state(int d_state, int headdim, const SsdStatePair& sp, int subs, int batch, hipStream_t st);

struct BwdArgs;
struct BwdPrepArgs;
struct BwdSumArgs;
bool bwd_supported(int d_state);
void bwd_segments(int d_inner, int batch, int seqlen, int* nseg, int* seg_len, int* seg_chunks);
void launch_bwd_prep(int io_bf16, const BwdPrepArgs& a, int sets, hipStream_t st);
hipError_t launch_bwd(int d_state, int io_bf16, const BwdArgs& a, int batch, hipStream_t st);   // (an error: nothing was launched)
void launch_bwd_sum(const BwdSumArgs& a, hipStream_t st);
}  // namespace bm
