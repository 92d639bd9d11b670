// view_order.h -- the order in which the backward kernel's passes over the views
// project, gather and use them.  Plain C++, so that the order is checked on the
// host.
#pragma once
#include <type_traits>
#include <utility>

#if defined(__HIPCC__)
#define QK_HD __host__ __device__ __forceinline__
#else
#define QK_HD inline
#endif

namespace qk {

// Calls f(integral_constant<int, K>) for K = B .. N - 1.
template <int B, int N, typename F>
QK_HD void static_for(F &&f) {
    if constexpr (B < N) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, N>(f);
    }
}

// The views 0 .. V - 1 in order, the taps of the next one in flight behind the
// current one.  proj(m0): lane K of a pixel's LPP lanes projects it into view m0 +
// K (the last view where there is none).  issue(K, m, slot): the taps of view m at
// lane K's projection into buffer slot; that projection is always view m's own, so
// its offsets lie in view m's map.  (Past the last view of a group cut short the
// last view's taps are asked for again: without the branch the gathers of a group
// stay one run; eight views of 270x480, C = 16: 748 us, 792 with it.)  step(m,
// slot): view m, in buffer slot.
template <int LPP, typename Proj, typename Issue, typename Step>
QK_HD void views_in_order(int V, Proj &&proj, Issue &&issue, Step &&step) {
    proj(0);
    issue(std::integral_constant<int, 0>{}, 0, std::integral_constant<int, 0>{});
    for (int m0 = 0; m0 < V; m0 += LPP) {
        static_for<0, LPP>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            const int m = m0 + k;
            if constexpr (k + 1 < LPP) {
                issue(std::integral_constant<int, k + 1>{}, m + 1 < V ? m + 1 : V - 1,
                      std::integral_constant<int, (k + 1) % 2>{});
            } else if (m + 1 < V) {
                proj(m + 1);
                issue(std::integral_constant<int, 0>{}, m + 1, std::integral_constant<int, (k + 1) % 2>{});
            }
            if (m < V) step(m, std::integral_constant<int, k % 2>{});
        });
    }
}

}  // namespace qk
