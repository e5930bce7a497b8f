// Host-side choices of librc (launch shapes, plans, strips) by their internal names, for tests
// that need no GPU. Each line of standard input is a command; each gives one line of output.
#include <cstdint>
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>

#include "kernels.h"
#include "runtime.h"

using namespace rc;

// demosaic <bilinear|gradient> images H W sectors: rows per band.
static void demosaic(std::istringstream& in) {
    std::string method;
    int images, H, W, sectors;
    in >> method >> images >> H >> W >> sectors;
    const int64_t band = method == "bilinear"
                             ? demosaic_band(images, H, W, sectors != 0, 256)
                             : demosaic_gradient_band(images, H, W, sectors != 0, 256);
    std::printf("%lld\n", (long long)band);
}

int main() {
    std::string line, cmd;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        in >> cmd;
        if (cmd == "demosaic") demosaic(in);
        else return 1;
        std::fflush(stdout);
    }
    return 0;
}
