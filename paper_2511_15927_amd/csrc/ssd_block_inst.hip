// Instantiations and launcher of the one-chunk Mamba-2 call (ssd_block.h).
#include "ssd_block.h"
#include "launch.h"

namespace bm {

static constexpr size_t kMaxLds = 160 * 1024;

template <int N, int BLOCKS>
static hipError_t prep_one(const SsdBlockArgs& a, hipStream_t st)
{
    static LdsLimit limit;
    constexpr size_t lds = ssd_block_prep_lds<N, BLOCKS>();
    auto prep = ssd_block_prep_kernel<N, BLOCKS>;
    if (lds > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(prep), lds);
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(prep, dim3((unsigned)a.G, 2, (unsigned)a.batch), dim3(1024), lds, st, a);
    return hipSuccess;
}

template <int N, bool COMMIT, bool SHARED>
static hipError_t whole_one(const SsdBlockArgs& a, dim3 grid, hipStream_t st)
{
    static LdsLimit limit;
    auto kernel = ssd_block_kernel<N, 1, COMMIT, SHARED, true>;
    const hipError_t err = limit.raise(reinterpret_cast<const void*>(kernel), kMaxLds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kernel, grid, dim3(1024), (SsdBlockLds<N, COMMIT, SHARED>::bytes(a.tiles)), st, a);
    return hipSuccess;
}

template <int N, int BLOCKS>
static hipError_t launch_one(const SsdBlockArgs& a, hipStream_t st)
{
    if constexpr (BLOCKS == 1) {
        if (a.tiles) {
            const dim3 grid((unsigned)((a.Dn + 64 * a.tiles - 1) / (64 * a.tiles)), 1, (unsigned)a.batch);
            if (a.h_out) return a.shared ? whole_one<N, true, true>(a, grid, st) : whole_one<N, true, false>(a, grid, st);
            return a.shared ? whole_one<N, false, true>(a, grid, st) : whole_one<N, false, false>(a, grid, st);
        }
    }
    const dim3 grid((unsigned)((a.Dn + 63) / 64), 1, (unsigned)a.batch);
    if (a.h_out) {
        if (a.shared) hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, true, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, true, false>), grid, dim3(256), 0, st, a);
    } else {
        if (a.shared) hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, false, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, false, false>), grid, dim3(256), 0, st, a);
    }
    return hipSuccess;
}

// Tiles of a workgroup where the call goes in one launch, else 0: as few as give every CU one workgroup at most.  Each workgroup
// makes the operands of its group for itself, which a second round of them would pay for again.  us, d_inner 4096, 32 tokens, 64
// x 64 heads, 128 states, state not committed (two launches; one launch with 1, 2, 3, 4 tiles):  batch 1 10.8; 8.0, 9.6, 11.4, 13.6
// 8 12.6; 15.4, 10.0, 11.8, 14.1   12 15.5; 22.5, 18.7, 22.7, 15.0   16 18.6; 30.0, 19.7, 23.6, 16.2   17 21.0; 36, 27, 23, 28
// 32 27.3; 58, 37, 35, 29.9.  d_inner 1024, 64 states: batch 1 11.7; 7.2   32 13.2; 13.5, 9.0, 9.9, 11.0.
// What a workgroup reads and holds for a second set of x leaves LDS for three tiles.
int ssd_block_tiles(int d_state, const SsdBlockArgs& a)
{
    if (a.L > 32) return 0;
    const long long tiles = (a.Dn + 63) / 64, group = (long long)a.HG * a.P;
    for (int n = 1; n <= 4; n++) {
        if (a.batch * ((tiles + n - 1) / n) > cu_count()) continue;
        const bool fits = (d_state == 128 ? (a.shared ? SsdBlockLds<128, true, true>::bytes(n) : SsdBlockLds<128, true, false>::bytes(n))
                                          : (a.shared ? SsdBlockLds<64, true, true>::bytes(n) : SsdBlockLds<64, true, false>::bytes(n))) <= kMaxLds;
        return fits && (a.G == 1 || group % (64 * n) == 0) ? n : 0;
    }
    return 0;
}

hipError_t launch_ssd_block(int d_state, const SsdBlockArgs& a, hipStream_t st)
{
    if (d_state == 128) return a.L <= 32 ? launch_one<128, 1>(a, st) : launch_one<128, 2>(a, st);
    return a.L <= 32 ? launch_one<64, 1>(a, st) : launch_one<64, 2>(a, st);
}

hipError_t launch_ssd_block_prep(int d_state, const SsdBlockArgs& a, hipStream_t st)
{
    if (d_state == 128) return a.L <= 32 ? prep_one<128, 1>(a, st) : prep_one<128, 2>(a, st);
    return a.L <= 32 ? prep_one<64, 1>(a, st) : prep_one<64, 2>(a, st);
}

}  // namespace bm
