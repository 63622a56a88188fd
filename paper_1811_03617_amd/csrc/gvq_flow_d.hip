// Instances of the decompress kernel of gvq_flow.h.
#include "gvq_flow.h"

flow_kernel gvq_flow_decompress(const FlowPlan& p)
{
    flow_kernel kern = nullptr;
    flow_decompress_instance(p, [&](auto kst, auto etw, auto exact, auto waves) {
        kern = decompress_flow_kernel<decltype(etw)::value, decltype(kst)::value, decltype(exact)::value, decltype(waves)::value>;
    });
    return kern;
}
