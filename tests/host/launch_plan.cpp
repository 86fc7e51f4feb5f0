// Host check of the workgroup shapes (launch_plan.hpp): the automatic shape
// given as options is planned as the automatic one, wholly or in part; any
// other shape stays the caller's.
#include <cstdio>

#include "launch_plan.hpp"

using namespace dtans;

int main() {
    int fails = 0;
    auto expect = [&](bool ok, const char *what, bool f64, bool row, int w, int g) {
        if (!ok) {
            ++fails;
            printf("%s: f64=%d row=%d waves=%d groups=%d\n", what, f64, row, w, g);
        }
    };
    for (int c = 0; c < 4; ++c) {
        const bool f64 = c & 1, row = c & 2;
        const ShapePlan a = plan_shape(f64, row, 0, 0);
        expect(!a.fixed && a.wg_per_cu == 2 && a.waves_per_wg == (row ? 16 : 12), "automatic", f64, row, 0, 0);
        for (int w = 0; w <= 16; ++w)
            for (int g = 0; g <= 32; ++g) {
                const ShapePlan p = plan_shape(f64, row, w, g);
                expect(!w || p.waves_per_wg == w, "waves kept", f64, row, w, g);
                expect(!g || p.wg_per_cu == g, "groups kept", f64, row, w, g);
                const bool same = p.waves_per_wg == a.waves_per_wg && p.wg_per_cu == a.wg_per_cu;
                expect(p.fixed == !same, "fixed", f64, row, w, g);
            }
    }
    printf("%d failures\n", fails);
    return fails != 0;
}
