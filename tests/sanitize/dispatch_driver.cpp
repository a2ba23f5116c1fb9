// The dispatch rules of spice_internal.h on layers read from stdin, one per line as
// "T d N K C I Is wfmt": prints the tile shape (0 Small, 1 Wide, 2 Big), the shared block's
// parts, whether the layer call's fused launches are the shorter, and whether the GEMM tiles are for
// the LoRE corrections alone.
#include <cstdio>

#include "spice_internal.h"

int main(int argc, char**) {
    if (argc > 1) {  // routing instead: "T N d dtype part_bytes x_to_host": contraction parts, row per wave
        int T, N, d, dtype, host;
        long bytes;
        while (std::scanf("%d %d %d %d %ld %d", &T, &N, &d, &dtype, &bytes, &host) == 6) {
            const int parts = spice::route_parts(T, N, d, dtype, (size_t)bytes);
            std::printf("%d %d\n", parts, spice::route_keeps_rows(T, N, d, parts, host != 0));
        }
        return 0;
    }
    int T, d, N, K, C, I, Is, wfmt;
    while (std::scanf("%d %d %d %d %d %d %d %d", &T, &d, &N, &K, &C, &I, &Is, &wfmt) == 8)
        std::printf("%d %d %d %d\n", spice::gemm_shape(T, N, K, C, I, Is, wfmt), spice::gemm_shared_parts(T, d, N, K, C, I, Is),
                    spice::layer_fused_is_shorter(T, d, N, K, Is), spice::lore_gemm_is_shorter(T, d, N, K));
}
