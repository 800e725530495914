// Prints the traversal's launch shapes (test infrastructure), a line per line
// read: "deals npix node_bytes tri_bytes" and
// "blocks cus cap bpc most deals" and "lds stack" (bytes of a block,
// blocks resident, blocks accepted).
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
        } else if (what == "lds") {
            std::cin >> a;
            printf("%d %d %d\n", neb::trace_lds_bytes((int)a), neb::trace_blocks_resident((int)a),
                   neb::trace_blocks_accepted((int)a));
        } else {
            std::cin >> a >> b >> c >> d >> e;
            printf("%d\n", neb::trace_blocks((int)a, b, (int)c, (int)d, e != 0));
        }
    }
    return 0;
}
