// The integer keys by which logits are ranked: in the order of the floats, both zeros alike, above the least integer.
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include "../../paper_2502_12224_amd/csrc/float_order.h"

int main() {
    const float inf = INFINITY, tiny = 1.4e-45f, least = 1.17549435e-38f;
    const float v[] = {-inf, -3.4e38f, -2.0f, -1.0f, -0.5f, -least, -tiny, -0.0f, 0.0f, tiny, least, 0.5f, 1.0f, 1.00000012f, 2.0f, 3.4e38f, inf};
    for (float a : v)
        for (float b : v) {
            const int ka = fate::float_order(a), kb = fate::float_order(b);
            if ((ka > kb) != (a > b) || (ka == kb) != (a == b) || ka == INT_MIN) {
                std::printf("float order: %g and %g have keys %d and %d\n", a, b, ka, kb);
                return 1;
            }
        }
    std::puts("float order driver: ok");
    return 0;
}
