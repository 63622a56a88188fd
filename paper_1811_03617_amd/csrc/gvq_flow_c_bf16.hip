// Instances of the compress kernel of gvq_flow.h for bf16 gradients.
#include "gvq_flow.h"

flow_kernel gvq_flow_compress_bf16(const FlowPlan& p)
{
    flow_kernel kern = nullptr;
    flow_compress_instance(p, [&](auto tiles, auto steps, auto exact, auto waves) {
        kern = compress_flow_kernel<decltype(tiles)::value, decltype(steps)::value, true, decltype(exact)::value, decltype(waves)::value>;
    });
    return kern;
}
