"""CPU: the cache update's division by a group's stored scale.  The kernel computes y / s
as q = y r, q + (y - q s) r with r = 1 / s rounded; this program compares it with the
IEEE division for every significand of s with 11 bits (binary16 scales; bfloat16 ones
are among them) and every 24-bit significand of y, 2^33 pairs, and counts how often the
product alone would differ.  Other exponents only shift both results, as long as nothing
is subnormal (the kernel's bounds keep to that)."""
import ctypes
import subprocess

SOURCE = r"""
#include <stdint.h>
#include <string.h>
static float bits(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static uint32_t word(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
/* scales first .. last - 1 of the 1024; bad[0]: three steps differ, bad[1]: y r differs */
void compare(int first, int last, int64_t *bad) {
  for (int i = first; i < last; ++i) {
    const float s = bits(0x3f800000u | (uint32_t)i << 13), r = 1.0f / s;
    for (uint32_t block = 0; block < 1u << 23; block += 1u << 12) {
      int32_t d0 = 0, d1 = 0;
      for (uint32_t m = block; m < block + (1u << 12); ++m) {
        const float y = bits(0x3f800000u | m), q = y * r, want = y / s;
        const float got = __builtin_fmaf(__builtin_fmaf(-q, s, y), r, q);
        d0 += word(got) != word(want);
        d1 += word(q) != word(want);
      }
      bad[0] += d0;
      bad[1] += d1;
    }
  }
}
"""


def test_three_step_division_is_the_ieee_division(tmp_path):
    from concurrent.futures import ThreadPoolExecutor
    src, lib = tmp_path / "div.c", tmp_path / "div.so"
    src.write_text(SOURCE)
    subprocess.run(["gcc", "-O3", "-march=native", "-ffp-contract=off", "-shared", "-fPIC", str(src), "-o", str(lib)],
                   check=True)
    fn = ctypes.CDLL(str(lib)).compare

    def part(i):
        bad = (ctypes.c_int64 * 2)()
        fn(i * 64, (i + 1) * 64, bad)
        return bad[0], bad[1]

    with ThreadPoolExecutor(8) as ex:
        counts = list(ex.map(part, range(16)))
    assert sum(c[0] for c in counts) == 0
    assert sum(c[1] for c in counts) > 0  # the comparison does see roundings that differ
