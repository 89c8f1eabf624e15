// gemm_plan: for "reduce pieces splits" lines on standard input the lanes that share a piece in a sum of slices.
#include <cstdio>
#include <cstring>

#include "fxp_gemm_plan.h"

int main() {
    char what[16];
    long long a, b;
    while (std::scanf("%15s %lld %lld", what, &a, &b) == 3) std::printf("%d\n", fxp::reduce_lanes(a, b));
}
