// Driver of tests/test_tagged_scalars.py: the hand-over of scalars from a kernel to the polling
// host (csrc/tagged.h), fed with every state that stores arriving line by line, in any order, can
// leave in host memory.
#include <cstdio>
#include <vector>

#include "tagged.h"

int main() {
    const int n = 20;   // five 64-byte lines
    std::vector<ba::Tagged> m(n);
    std::vector<double> out(n);
    int accepted = 0;
    for (int arrived = 0; arrived < 32; ++arrived) {
        for (int i = 0; i < n; ++i) {
            const bool there = arrived >> (i / 4) & 1;
            m[i] = there ? ba::Tagged{100.0 + i, 8.0} : ba::Tagged{double(i), 7.0};
        }
        if (!ba::tagged_read(m.data(), n, 8.0, out.data())) continue;
        ++accepted;
        for (int i = 0; i < n; ++i)
            if (out[i] != 100.0 + i) {
                std::printf("a value of the last hand-over: lines %d, value %d\n", arrived, i);
                return 1;
            }
    }
    std::printf("accepted %d of 32\n", accepted);
    return accepted == 1 ? 0 : 1;
}
