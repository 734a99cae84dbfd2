// Which kernel the router's launch code picks for shapes read from stdin ("bf16|f32 T H E k"),
// on a device of 256 CUs: the launch code of route.hip compiled for the host, with launches
// recorded and not run.
#include <hip/hip_runtime.h>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) record(kernel, __VA_ARGS__)

template <typename K, typename... A>
void record(K kernel, A... args);

#include "../../paper_2608_21614_amd/csrc/route.hip"

using namespace saem;

struct Known {
    const void* kernel;
    const char* name;
};
template <typename Elt>
std::vector<Known> known() {
    return {{(const void*)&k_router_scores<Elt, 1, 1, true>, "1,1,true"},   {(const void*)&k_router_scores<Elt, 2, 1, true>, "2,1,true"},
            {(const void*)&k_router_scores<Elt, 4, 1, true>, "4,1,true"},   {(const void*)&k_router_scores<Elt, 2, 2, true>, "2,2,true"},
            {(const void*)&k_router_scores<Elt, 4, 2, true>, "4,2,true"},   {(const void*)&k_router_scores<Elt, 4, 2, false>, "4,2,false"},
            {(const void*)&k_router_scores<Elt, 4, 1, false>, "4,1,false"}, {(const void*)&k_router_scores<Elt, 2, 1, false>, "2,1,false"},
            {(const void*)&k_router_scores<Elt, 1, 1, false>, "1,1,false"}};
}

template <typename K, typename... A>
void record(K kernel, A... args) {
    const long long v[] = {(long long)(size_t)0, [](auto a) -> long long {
                               if constexpr (std::is_integral_v<decltype(a)>) return a;
                               else return 0;
                           }(args)...};
    for (const Known& k : known<uint16_t>())
        if (k.kernel == (const void*)kernel) printf(" bf16:%s:%lld", k.name, v[4]);  // rows
    for (const Known& k : known<float>())
        if (k.kernel == (const void*)kernel) printf(" f32:%s:%lld", k.name, v[4]);
}

int main() {
    char dtype[8];
    Shape s{};
    while (scanf("%7s %d %d %d %d", dtype, &s.T, &s.H, &s.E, &s.k) == 5) {
        s.bf16 = dtype[0] == 'b';
        if (launch_route_topk(s, nullptr, nullptr, nullptr, nullptr, false, nullptr, nullptr, nullptr, nullptr)) return 1;
        printf("\n");
    }
    printf("all");
    for (const char* dt : {"bf16", "f32"})
        for (const Known& k : known<float>()) printf(" %s:%s", dt, k.name);
    printf("\n");
    return 0;
}
