// Instances of the decompress kernel of gvq_flow.h.
#include "gvq_flow.h"

flow_kernel gvq_flow_decompress(const FlowPlan& p, bool exact)
{
    auto exact4 = [](auto t, auto s) -> flow_kernel { return decompress_flow_kernel<decltype(s)::value, decltype(t)::value, true, 4>; };
    auto split4 = [](auto t, auto s) -> flow_kernel { return decompress_flow_kernel<decltype(s)::value, decltype(t)::value, false, 4>; };
    auto exact8 = [](auto t, auto s) -> flow_kernel { return decompress_flow_kernel<decltype(s)::value, decltype(t)::value, true, 8>; };
    auto split8w = [](auto t, auto s) -> flow_kernel { return decompress_flow_kernel<decltype(s)::value, decltype(t)::value, false, 8>; };
    if (p.waves == 8) {
        if (exact) return p.kst == 1 ? flow_pick<1>(p.etw, FlowSteps<7, 8>{}, exact8) : nullptr;
        if (p.kst == 2) return flow_pick<2>(p.etw, FlowSteps<5, 6, 7, 8>{}, split8w);
        if (p.kst == 3) return flow_pick<3>(p.etw, FlowSteps<3, 4, 5, 6, 7>{}, split8w);
        return p.kst == 4 ? flow_pick<4>(p.etw, FlowSteps<3, 4, 5>{}, split8w) : nullptr;
    }
    if (exact) {
        // fewer than 10 flop/B: more than 32 comps only with slices of at most 40
        if (p.kst == 1) return flow_pick<1>(p.etw, FlowSteps<1, 2, 3, 4, 5, 6, 7, 8, 10, 12>{}, exact4);
        return p.kst == 2 ? flow_pick<2>(p.etw, FlowSteps<1>{}, exact4) : nullptr;
    }
    if (p.kst == 1) return flow_pick<1>(p.etw, FlowSteps<1, 2, 3, 4, 5, 6, 7, 8, 10, 12>{}, split4);
    if (p.kst == 2) return flow_pick<2>(p.etw, FlowSteps<1, 2, 3, 4, 5, 6, 7, 8>{}, split4);
    if (p.kst == 3) return flow_pick<3>(p.etw, FlowSteps<1, 2, 3, 4, 5>{}, split4);
    return p.kst == 4 ? flow_pick<4>(p.etw, FlowSteps<1, 2, 3, 4>{}, split4) : nullptr;
}
