// Instances of the compress kernel of gvq_flow.h for f32 gradients.
#include "gvq_flow.h"

flow_kernel gvq_flow_compress_f32(const FlowPlan& p, bool exact)
{
    auto exact4 = [](auto t, auto s) -> flow_kernel { return compress_flow_kernel<decltype(t)::value, decltype(s)::value, false, true, 4>; };
    auto split4 = [](auto t, auto s) -> flow_kernel { return compress_flow_kernel<decltype(t)::value, decltype(s)::value, false, false, 4>; };
    auto split8w = [](auto t, auto s) -> flow_kernel { return compress_flow_kernel<decltype(t)::value, decltype(s)::value, false, false, 8>; };
    if (p.waves == 8) {
        if (p.ntw != 1) return nullptr;
        return exact ? nullptr : flow_pick<1>(p.steps, FlowSteps<10, 12, 16>{}, split8w);
    }
    if (exact) {
        // fewer than 10 flop/B: more than 16 comps only with short slices
        if (p.ntw == 1) return flow_pick<1>(p.steps, FlowSteps<1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16>{}, exact4);
        if (p.ntw == 2) return flow_pick<2>(p.steps, FlowSteps<1, 2, 3, 4>{}, exact4);
        return p.ntw == 3 ? flow_pick<3>(p.steps, FlowSteps<1, 2>{}, exact4) : nullptr;
    }
    if (p.ntw == 1) return flow_pick<1>(p.steps, FlowSteps<2, 3, 4, 5, 6, 7, 8, 10, 12, 16>{}, split4);
    if (p.ntw == 2) return flow_pick<2>(p.steps, FlowSteps<2, 3, 4, 5, 6, 7, 8>{}, split4);
    if (p.ntw == 3) return flow_pick<3>(p.steps, FlowSteps<2, 3, 4, 5>{}, split4);
    return p.ntw == 4 ? flow_pick<4>(p.steps, FlowSteps<2, 3, 4>{}, split4) : nullptr;
}
