// topk_emit with attention that gathers K and V rows (sketch and RAW scores),
// from one cache or (at.loc) from the two pools of a tiered one.
#include "topk_device.h"

namespace hill {

namespace {

template <int DT, bool STREAM>
void emit(const RefineArgs& r, const AttnArgs& at, hipStream_t st, Stamp ts)
{
    if (at.loc) emit_attn_gc<DT, STREAM, false, true>(r, at, st, ts);
    else emit_attn_gc<DT, STREAM, false>(r, at, st, ts);
}

}  // namespace

hipError_t launch_emit_gather(const RefineArgs& r, const AttnArgs& at, int dtype, bool streamed, hipStream_t st, Stamp ts)
{
    if (dtype == 1) {
        if (streamed) emit<1, true>(r, at, st, ts);
        else emit<1, false>(r, at, st, ts);
    } else {
        if (streamed) emit<0, true>(r, at, st, ts);
        else emit<0, false>(r, at, st, ts);
    }
    return hipGetLastError();
}

}  // namespace hill
