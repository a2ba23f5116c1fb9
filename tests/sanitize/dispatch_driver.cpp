// The GEMM dispatch rules of spice_internal.h on layers read from stdin, one per line as
// "T d N K C I Is wfmt": prints the tile shape (0 Small, 1 Wide, 2 Big), the shared block's
// parts, whether the layer call's fused launches are the shorter, and whether the GEMM tiles are for
// the LoRE corrections alone.
#include <cstdio>

#include "spice_internal.h"

int main() {
    int T, d, N, K, C, I, Is, wfmt;
    while (std::scanf("%d %d %d %d %d %d %d %d", &T, &d, &N, &K, &C, &I, &Is, &wfmt) == 8)
        std::printf("%d %d %d %d\n", spice::gemm_shape(T, N, K, C, I, Is, wfmt), spice::gemm_shared_parts(T, d, N, K, C, I, Is),
                    spice::layer_fused_is_shorter(T, d, N, K, Is), spice::lore_gemm_is_shorter(T, d, N, K));
}
