"""Places of keys in the emission (CPU): the function that the kernel uses,
compiled for the host, against 64-bit arithmetic, with blocks and primitives
that begin on either side of 2^32 keys."""
import os
import random
import subprocess

import pytest

from paper_2508_03180_amd import build as hipbuild

MAIN = """
#include <stdio.h>
#include "common.h"
int main() {
    unsigned b, o, k;
    while (scanf("%u %u %u", &b, &o, &k) == 3) printf("%u\\n", dgs::key_place(b, o, k));
}
"""
EMIT_KEYS = 2048       # keys of a workgroup
MAX_KEYS = 1 << 30     # key capacity
BLOCK = 1024 * 2 ** 22  # keys of a block of primitives that each cover 2^22 tiles


@pytest.mark.skipif(not os.path.exists(hipbuild.HIPCC), reason="needs hipcc")
def test_places(tmp_path):
    src, exe = tmp_path / "place.hip", str(tmp_path / "place")
    src.write_text(MAIN)
    subprocess.check_call([hipbuild.HIPCC, *hipbuild.FLAGS, str(src), "-o", exe], stderr=subprocess.DEVNULL)
    rng = random.Random(1)
    cases = [(0, 0, 0), (2048, 5, 2048), (2 ** 32 - 1, 0, 0), (2 ** 32 - 1, 7, 6), (2 ** 32 - 4, 8, 0)]
    for _ in range(3000):
        k0 = rng.randrange(MAX_KEYS // EMIT_KEYS) * EMIT_KEYS
        start = rng.choice([rng.randrange(2 * MAX_KEYS), 2 ** 32 - 1 - rng.randrange(5000), rng.randrange(2 ** 32),
                            rng.randrange(2 ** 36)])  # keys before the block
        off = rng.choice([rng.randrange(5000), rng.randrange(BLOCK), k0 + 1 + rng.randrange(EMIT_KEYS)])
        cases.append((start, off, k0))
    text = "".join(f"{min(b, 2 ** 32 - 1)} {o} {k}\n" for b, o, k in cases)
    got = [int(x) for x in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()]
    assert len(got) == len(cases)
    inside = 0
    for (b, o, k), g in zip(cases, got):
        true = b + o - k
        if 0 <= true < EMIT_KEYS:  # the workgroup's keys
            assert g == true, (b, o, k)
            inside += 1
        else:
            assert g >= EMIT_KEYS, (b, o, k, g)
    assert inside > 0
