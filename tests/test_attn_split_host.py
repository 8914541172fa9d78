"""How attention cuts a sequence's keys (csrc/attn_split.h), compiled for the host: every split that poss_set_tuning or the rule can
ask for, up to the longest context, stays within what the kernels hold - a page-table entry per lane, 64 blocks a split, and 256 splits -
and is the split asked for wherever that fits, the same for every size of the tree region."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "attn_split.h"
#include <stdio.h>
using namespace poss;
static long wrong = 0, cut = 0;
static void check(int prefix, int region, int keys) {
    const int n_blocks = (prefix + region + 31) / 32, most = (prefix + 128 + 31) / 32, bps = attn_blocks_per_split(prefix, keys);
    const int n_splits = bps > 0 ? (n_blocks + bps - 1) / bps : 0;
    bool ok = bps >= 1 && bps <= 64 && n_splits >= 1 && n_splits <= 256;
    const int asked = keys / 32 < 64 ? keys / 32 : 64;
    if (keys > 0 && (most + asked - 1) / asked <= 256) ok = ok && bps == asked; else if (keys > 0) ++cut;
    if (!ok && wrong++ < 5) printf("prefix %d region %d keys per split %d: %d blocks per split, %d splits\n", prefix, region, keys, bps, n_splits);
}
int main() {
    for (int keys = -512; keys <= 20000; keys += keys < 0 ? 512 : keys == 0 ? 64 : 32)
        for (int region = 1; region <= 128; region += 127)
            for (int prefix = 0; prefix <= 500000; prefix = prefix < 500000 && prefix + 997 > 500000 ? 500000 : prefix + 997) {
                check(prefix, region, keys);
                const int edge = (prefix + region + 31) / 32 * 32 - region;      // the last key of a block, and the first of the next
                if (edge < 500000) { check(edge, region, keys); check(edge + 1, region, keys); }
            }
    printf("wrong %ld, cut %ld\n", wrong, cut);
    return wrong || !cut;
}
"""


def test_splits_fit_the_kernels(tmp_path):
    src, exe = tmp_path / "split.cc", tmp_path / "split"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2506_03566_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    print(r.stdout)
    assert r.returncode == 0
