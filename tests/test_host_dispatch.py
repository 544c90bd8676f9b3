"""The rules that choose a hop kernel (no GPU), compiled for the host from the
library's own header."""
import math
import subprocess

import pytest

from paper_1804_08593_amd import build

# precision, Ls, with the fused update, workgroups of the small-launch kernel, chosen
LINES = [
    ("F64", 8, 0, 512, 1), ("F64", 8, 1, 656, 1), ("F64", 12, 1, 640, 1),
    ("F64", 16, 0, 512, 1), ("F64", 16, 0, 513, 0), ("F64", 16, 1, 640, 0), ("F64", 20, 1, 683, 0),
    ("F64", 24, 0, 512, 1), ("F64", 24, 1, 640, 0), ("F64", 32, 0, 256, 1), ("F64", 32, 1, 320, 0),
    ("F32", 16, 1, 640, 1), ("F32", 20, 0, 683, 1), ("F32", 24, 0, 768, 1), ("F32", 24, 1, 800, 0),
    ("F32", 32, 0, 512, 1), ("F32", 32, 1, 640, 0),
    ("F16", 16, 0, 640, 1), ("F16", 16, 1, 512, 1), ("F16", 16, 1, 576, 0), ("F16", 8, 1, 640, 0),
    ("F16", 20, 0, 683, 1), ("F16", 24, 0, 800, 0), ("F16", 32, 0, 640, 0),
]


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src = d / "rules.hip"
    src.write_text('''#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "kernels.h"
using namespace mspcg;
template <class S> static void line(long vh, int Ls, int ndom, int cg) {
    printf("%d %ld %ld\\n", (int)hop_is_small<S>(vh, Ls, ndom, cg), hop_grid_x<S>(vh, Ls, ndom, true, cg),
           hop_grid_x<S>(vh, Ls, ndom, false, cg));
}
int main(int n, char** v) {
    if (!strcmp(v[1], "rows")) {  // outputs, block, largest box, domains
        for (int i = 2; i + 3 < n; i += 4)
            printf("%d\\n", (int)hop_is_rows<F16>(atol(v[i]), atol(v[i + 1]), atol(v[i + 2]), 16, atoi(v[i + 3])));
        return 0;
    }
    for (int i = 1; i + 4 < n; i += 5) {
        const long vh = atol(v[i + 1]);
        const int Ls = atoi(v[i + 2]), nd = atoi(v[i + 3]), cg = atoi(v[i + 4]);
        if (!strcmp(v[i], "F64")) line<F64>(vh, Ls, nd, cg);
        else if (!strcmp(v[i], "F32")) line<F32>(vh, Ls, nd, cg);
        else line<F16>(vh, Ls, nd, cg);
    }
}
''')
    exe = d / "rules"
    r = subprocess.run(["hipcc", "-std=c++17", "-O1", "--cuda-host-only", "-I", build.CSRC, str(src),
                        "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(cases):
        args = [str(x) for c in cases for x in c]
        out = subprocess.run([str(exe), *args], capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in ln.split()) for ln in out.splitlines()]
    return run


def test_small_launch_hop_is_chosen_by_resident_workgroups(rules):
    got = rules([(p, wg * (64 // ls), ls, 1, cg) for p, ls, cg, wg, _ in LINES])
    for (p, ls, cg, wg, want), (small, gx, gen) in zip(LINES, got):
        assert small == want, (p, ls, cg, wg)
        assert gen == -(-wg * (64 // ls) // (256 // ls))
        assert gx == (wg if want else gen)


def test_small_launch_hop_counts_every_domain(rules):
    # 16 domains of 33 workgroups each against one domain of as many sites
    for p, ls, cg in (("F64", 16, 0), ("F16", 16, 1)):
        (a, _, _), (b, _, _), (c, _, _) = rules([(p, 32 * 4, ls, 16, cg), (p, 32 * 4 + 1, ls, 16, cg),
                                                 (p, 32 * 4 * 16, ls, 1, cg)])
        assert (a, b, c) == (1, 0, 1)
    # never beyond 42000 entries
    assert rules([("F32", 5251, 8, 1, 0), ("F32", 5250, 8, 1, 0)]) == [(0, 165, 165), (1, 657, 165)]


def _boxes(dims, block, pad=2):
    """Sites of one parity: widened by 1, the block, widened by pad; domains."""
    def vol(k):
        return math.prod(L if L == b else b + 2 * k for L, b in zip(dims, block)) // 2
    return vol(min(pad, 1)), vol(0), vol(pad), math.prod(L // b for L, b in zip(dims, block))


@pytest.mark.parametrize("dims,block,pad,want", [
    ((24, 24, 24, 24), (12, 12, 12, 12), 2, 1), ((24, 24, 24, 48), (12, 12, 12, 24), 2, 1),
    ((24, 24, 24, 48), (24, 12, 24, 48), 2, 1), ((24, 24, 24, 24), (24, 24, 24, 24), 2, 1),
    ((16, 24, 28, 32), (4, 12, 14, 16), 2, 1), ((24, 24, 24, 24), (4, 4, 4, 4), 0, 1),
    # most of the widened blocks is rim
    ((24, 24, 24, 24), (8, 8, 8, 8), 2, 0), ((24, 24, 24, 24), (6, 6, 6, 6), 2, 0),
    ((48, 16, 16, 16), (12, 8, 8, 8), 2, 0), ((24, 24, 24, 24), (24, 6, 6, 6), 2, 0),
    ((24, 24, 24, 48), (4, 4, 4, 4), 2, 0), ((16, 16, 16, 32), (4, 4, 4, 8), 2, 0),
    # too few sites in the blocks themselves
    ((20, 20, 20, 20), (10, 10, 10, 10), 2, 0), ((16, 16, 16, 32), (8, 8, 8, 8), 2, 0),
    ((32, 8, 8, 64), (16, 4, 4, 32), 2, 0),
    # too few outputs
    ((16, 16, 16, 40), (16, 16, 16, 20), 2, 0),
], ids=str)
def test_matrix_core_hop_is_chosen_where_blocks_fill_their_boxes(rules, dims, block, pad, want):
    out, inner, widest, nd = _boxes(dims, block, pad)
    assert rules([("rows", out, inner, widest, nd)]) == [(want,)]
