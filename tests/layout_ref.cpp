// Prints samplers_beside_streaming for "cus lds" pairs read from stdin.
#include <cstdio>

#include "../paper_2609_21858_amd/csrc/psd_layout.hpp"

int main() {
    int cus;
    long lds;
    while (std::scanf("%d %ld", &cus, &lds) == 2) std::printf("%ld\n", psd::samplers_beside_streaming(cus, (size_t)lds));
}
