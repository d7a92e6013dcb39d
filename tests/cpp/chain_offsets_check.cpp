// Addresses of the chained products in blocks of more than 2^32 bytes: the
// 64-bit first element of a tile, chunk and segment plus a lane's 32-bit byte
// offset from it is the element, at the far corner of the block.
#include <cstdio>
#include <initializer_list>

#include "kernels.h"

namespace {
int failures = 0;
void check(bool ok, const char* what, int lay) {
    if (ok) return;
    ++failures;
    std::printf("wrong: %s, layout %d\n", what, lay);
}
// what a lane reads: base + unsigned(8 i), i in 32 bits
long long lane(long long base, unsigned i) { return 8 * base + (long long)(8u * i); }
}  // namespace

int main() {
    const int n = 30000, tile = 16 * 8, chunk = 32;  // 7.2 GB of FP64 values
    const long long off = 12345;
    check(spk::chain_lanes_fit(n), "block accepted", -1);
    check(!spk::chain_lanes_fit(1 << 22), "block wider than a lane's reach refused", -1);
    const int r0 = n - tile, k0 = n - chunk;  // first row or column of the last tile, first value of the last chunk
    for (int lay : {spk::kChainHeff, spk::kChainEnvL, spk::kChainEnvR})
        for (int r = 0; r < tile; ++r)
            for (int k = 0; k < chunk; ++k) {
                const long long row = r0 + r, val = k0 + k;
                // P(m, kc): rows of kc (left environments) or of m
                const bool pt = lay == spk::kChainEnvL, at = lay == spk::kChainHeff;
                check(lane(spk::chain_p(lay, off, n, r0, k0), pt ? unsigned(k * n + r) : unsigned(r * n + k)) ==
                          8 * (off + (pt ? val * n + row : row * n + val)),
                      "P", lay);
                // A(kc, kj), kc the tile's rows
                check(lane(spk::chain_a(lay, off, n, r0, k0), at ? unsigned(k * n + r) : unsigned(r * n + k)) ==
                          8 * (off + (at ? val * n + row : row * n + val)),
                      "A", lay);
                // B(kj, n), n the tile's columns
                check(lane(spk::chain_b(lay, off, n, k0, r0), pt ? unsigned(k * n + r) : unsigned(r * n + k)) ==
                          8 * (off + (pt ? val * n + row : row * n + val)),
                      "B", lay);
                if (failures > 20) return 1;
            }
    static_assert(sizeof(spk::KPrep::nd) == 8 && sizeof(spk::KPrep::nr) == 8, "site vectors of more than 2^31 values");
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
