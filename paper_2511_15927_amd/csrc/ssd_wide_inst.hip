// Launcher of the many-wave chunk walk (ssd_wide.h) for one (BM_N, BM_P), set on the command line.
#include "ssd_wide.h"
#include "launch.h"

namespace bm {

template <int HEADS, int MODE, int FORM>
static hipError_t variant(const SsdStatePair& sp, int batch, hipStream_t st)
{
    static LdsLimit limit;
    using W = SsdWide<BM_N, BM_P, HEADS>;
    auto kernel = ssd_wide_kernel<BM_N, BM_P, HEADS, MODE, FORM>;
    if (W::bytes() > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(kernel), W::bytes());
        if (err != hipSuccess) return err;
    }
    const unsigned parts = FORM == kSsdMeet ? 2u : FORM != kSsdWhole ? (unsigned)sp.dir[0].parts : 1u;
    const dim3 grid((unsigned)(sp.dir[0].H / HEADS), MODE == kSsdFinalOnly ? 2u * parts : parts, (unsigned)batch), block(W::kThreads);
    if constexpr (MODE == kSsdFinalOnly || FORM == kSsdMeet) hipLaunchKernelGGL(kernel, grid, block, W::bytes(), st, sp);
    else hipLaunchKernelGGL(kernel, grid, block, W::bytes(), st, sp.dir[0]);
    return hipSuccess;
}

template <int HEADS, int FORM>
static hipError_t launch(const SsdStatePair& sp, int dirs, int batch, hipStream_t st)
{
    if constexpr (FORM != kSsdMeet)
        if (dirs == 2) return variant<HEADS, kSsdFinalOnly, FORM>(sp, batch, st);
    switch (sp.dir[0].mode) {
        case kSsdPartial: return variant<HEADS, kSsdPartial, FORM>(sp, batch, st);
        case kSsdPartialRaw: return variant<HEADS, kSsdPartialRaw, FORM>(sp, batch, st);
        case kSsdFinalAdd: return variant<HEADS, kSsdFinalAdd, FORM>(sp, batch, st);
        default: return variant<HEADS, kSsdFinalAddRaw, FORM>(sp, batch, st);
    }
}

#define BM_NAME2(n, p) launch_ssd_wide_n##n##_p##p
#define BM_NAME(n, p) BM_NAME2(n, p)

// Two heads to a workgroup once one head each would not fit the chip at once: they share the tiles of their group.
hipError_t BM_NAME(BM_N, BM_P)(const SsdStatePair& sp, int dirs, int batch, hipStream_t st)
{
    const SsdArgs& sa = sp.dir[0];
    if (sa.meet) return launch<1, kSsdMeet>(sp, dirs, batch, st);
    if (sa.far) return launch<1, kSsdFarParts>(sp, dirs, batch, st);
    if (sa.parts > 1) return launch<1, kSsdParts>(sp, dirs, batch, st);
    if (sa.HG % 2 == 0 && (long long)sa.H * batch * dirs > cu_count()) return launch<2, kSsdWhole>(sp, dirs, batch, st);
    return launch<1, kSsdWhole>(sp, dirs, batch, st);
}

}  // namespace bm
