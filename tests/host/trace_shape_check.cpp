// Prints the traversal's launch shapes (test infrastructure), a line per line
// read: "deals npix node_bytes tri_bytes" and
// "blocks cus cap bpc most deals".
#include <cstdio>
#include <iostream>
#include <string>

#include "neb_trace_shape.h"

int main() {
    std::string what;
    while (std::cin >> what) {
        long long a, b, c, d, e;
        if (what == "deals") {
            std::cin >> a >> b >> c;
            printf("%d\n", (int)neb::trace_deals(a, b, c));
        } else {
            std::cin >> a >> b >> c >> d >> e;
            printf("%d\n", neb::trace_blocks((int)a, b, (int)c, (int)d, e != 0));
        }
    }
    return 0;
}
