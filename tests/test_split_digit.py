"""The split pass's digit of a key (CPU, the kernels' own code compiled for the host): where a tile
ranks its keys and where it writes them out it is the same, and inside the digit tables, for every
64-bit word; after a front end that gave up its bounded wait the keys are whatever memory held."""
import subprocess
import tempfile
from pathlib import Path

from paper_2608_15785_amd import build

SOURCE = r"""
#include "k_sort.hip"
#include <cstdio>
int main() {
    using namespace rgs;
    uint64_t x = 88172645463325252ull;
    long bad = 0;
    for (int i = 0; i < 200000; ++i) {
        x ^= x << 13, x ^= x >> 7, x ^= x << 17;
        for (uint32_t tile_bits = 0; tile_bits <= 10; ++tile_bits)
            for (uint32_t bits : {8u, 10u}) {
                const uint32_t shift = 32 + tile_bits, mask = (1u << bits) - 1;
                const PairsOut<uint64_t> out{nullptr, LocalKey{32, tile_bits}, nullptr};
                bad += out.digit(out.hold(x), shift, mask) != ((uint32_t)(x >> shift) & mask);
                const PairsOut<uint32_t> out32{nullptr, LocalKey{32 - bits, 0}, nullptr};
                bad += out32.digit(out32.hold((uint32_t)x), 32 - bits, mask) != ((uint32_t)x >> (32 - bits));
            }
    }
    std::printf("%ld\n", bad);
}
"""


def test_digit_of_any_word_is_the_ranked_one():
    with tempfile.TemporaryDirectory() as d:
        src, exe = Path(d) / "digit.hip", Path(d) / "digit"
        src.write_text(SOURCE)
        flags = [f for f in build.COMMON if f != "-fPIC"]
        subprocess.run([build.hipcc(), *flags, str(src), "-o", str(exe)], check=True, capture_output=True)
        assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.strip() == "0"
