// Plays the backward kernel's view order and follows which view each lane's
// projection and each tap buffer belongs to.
#include <cstdio>

#include "view_order.h"

static int fails = 0;
#define CHECK(c) do { if (!(c)) { std::printf("LPP %d, %d views: " #c "\n", LPP, V); ++fails; } } while (0)

template <int LPP>
static void check(int V) {
    int projected[LPP], buffer[2] = {-1, -1}, issued[16] = {}, used[16] = {}, last = -1;
    for (int &v : projected) v = -1;
    qk::views_in_order<LPP>(
        V,
        [&](int m0) {
            for (int k = 0; k < LPP; ++k) projected[k] = m0 + k < V ? m0 + k : V - 1;
        },
        [&](auto kk, int m, auto slot) {
            CHECK(m >= 0 && m < V);
            CHECK(projected[decltype(kk)::value] == m);   // offsets of a map used with that map
            buffer[decltype(slot)::value] = m;
            ++issued[m];
        },
        [&](int m, auto slot) {
            CHECK(m == last + 1);
            CHECK(buffer[decltype(slot)::value] == m);
            last = m;
            ++used[m];
        });
    CHECK(last == V - 1);
    for (int m = 0; m < V; ++m) CHECK(issued[m] >= 1 && used[m] == 1);
}

int main() {
    for (int V = 1; V <= 16; ++V) {
        check<2>(V);
        check<4>(V);
    }
    std::printf("%d failures\n", fails);
    return fails != 0;
}
