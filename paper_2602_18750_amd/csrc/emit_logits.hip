// topk_emit with attention whose logits are the scan's own (16-bit keys, ATTN
// scores): only V rows are gathered.
#include "topk_device.h"

namespace hill {

namespace {

template <int DT>
void emit(const RefineArgs& r, const AttnArgs& at, bool streamed, hipStream_t st, Stamp ts)
{
    if (streamed) emit_attn_gc<DT, true, true>(r, at, st, ts);
    else emit_attn_gc<DT, false, true>(r, at, st, ts);
}

}  // namespace

hipError_t launch_emit_logits(const RefineArgs& r, const AttnArgs& at, int dtype, bool streamed, hipStream_t st, Stamp ts)
{
    if (dtype == 1) emit<1>(r, at, streamed, st, ts);
    else emit<0>(r, at, streamed, st, ts);
    return hipGetLastError();
}

}  // namespace hill
