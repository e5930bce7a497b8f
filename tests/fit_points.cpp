// The calibration fit's device code run on the host over the most points its entry point takes
// (2^31 - 1, one detector, order 0): samples of 0, read through a stride of 0, and targets of 1,
// from one page mapped again and again. Prints the coefficients.
#include <sys/mman.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>

#include <hip/hip_runtime.h>

#include <algorithm>

// What the kernel's launch needs, unused here: this is a host program.
using std::min;
static const dim3 blockIdx, blockDim, threadIdx, gridDim;
#define __launch_bounds__(n)
#define hipLaunchKernelGGL(k, ...) (void)(k)
#include "fit.hip"

int main(int, char** argv) {
    const int points = std::atoi(argv[1]);
    // The targets: a file of ones, mapped as often as it takes.
    const size_t piece = (size_t)1 << 26, bytes = (size_t)points * 8;
    const int fd = memfd_create("ones", 0);
    if (fd < 0 || ftruncate(fd, piece) != 0) return 2;
    double* ones = (double*)mmap(nullptr, piece, PROT_READ | PROT_WRITE, MAP_SHARED, fd, 0);
    if (ones == MAP_FAILED) return 2;
    for (size_t i = 0; i < piece / 8; ++i) ones[i] = 1.0;
    char* y = (char*)mmap(nullptr, bytes + piece, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (y == MAP_FAILED) return 2;
    for (size_t at = 0; at < bytes; at += piece)
        if (mmap(y + at, piece, PROT_READ, MAP_SHARED | MAP_FIXED, fd, 0) == MAP_FAILED) return 2;
    const double x[1] = {0.0};
    double a[4] = {-1.0, -1.0, -1.0, -1.0};
    rc::fit_one<0>(x, (const double*)y, 0, 0, points, 0, a);
    std::printf("%g %g %g %g\n", a[0], a[1], a[2], a[3]);
    return 0;
}
