"""mspcg_apply's host path (no GPU): compiled with counting stubs for the launches and an
arena that holds a given number of intermediate fields, as mspcg_apply_noalloc uses it.
Where a field is missing the call is MSPCG_ENOMEM before anything is launched."""
import subprocess

from paper_1804_08593_amd import build, mspcg

# one-parity fields that each operator needs
FIELDS = {mspcg.OP_D: 4, mspcg.OP_DDAG: 2, mspcg.OP_HOP: 2, mspcg.OP_HOPDAG: 2, mspcg.OP_MHAT: 3,
          mspcg.OP_MHATDAG: 2, mspcg.OP_A: 5, mspcg.OP_M5INV: 0, mspcg.OP_PREPARE: 4}

SOURCE = r'''
#include <stdio.h>
#include "ctx.h"
namespace mspcg {
static int launches = 0;
template <> int launch_hop<F64>(const HopArgs<F64>&, int, int, bool, bool, hipStream_t, const HopReach*) { return ++launches, 0; }
template <> int launch_pack_prog<F64>(const double2*, const Field<F64>*, const Field<F64>*, const FiveDProg&, double, const int*, int, int, int, hipStream_t) { return ++launches, 0; }
template <> int launch_prog_full<F64>(const double2*, double2*, const FiveDProg&, double, const int*, int, hipStream_t) { return ++launches, 0; }
template <> int launch_unpack_parity<F64>(CField<F64>, double2*, const int*, int, int, int, hipStream_t) { return ++launches, 0; }
}
#include "api.hip"
int main() {
    static double2 field[2][4096];
    static char space[16 * 8192];
    for (int overlap = 0; overlap < 2; ++overlap)
        for (int op = 0; op <= MSPCG_OP_PREPARE; ++op)
            for (int k = 0; k <= 8; ++k) {
                mspcg_ctx c{};
                for (int m = 0; m < 4; ++m) c.L[m] = c.lat.E[m] = 2;
                c.Ls = 2, c.V4 = 16, c.Vh = c.lat.Vh = 8, c.Nh = 16;
                c.act.b = 1.5, c.act.c = 0.5, c.act.mf = 0.1;
                c.pr = make_progs(c.act, 4.3, 0.1);
                c.arena = space;
                c.arena_cap = (size_t)k * 16 * 12 * sizeof(double2);
                launches = 0;
                const int e = apply_op(&c, op, MSPCG_FP64, field[0], overlap ? field[0] + 12 : field[1], 0);
                printf("%d %d %d %d %d\n", overlap, op, k, e, launches);
            }
}
'''


def test_missing_fields_are_reported_before_any_launch(tmp_path):
    src, exe = tmp_path / "apply.hip", tmp_path / "apply"
    src.write_text(SOURCE)
    r = subprocess.run(["hipcc", "-std=c++17", "-O1", "--cuda-host-only", "-I", build.CSRC, str(src),
                        "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout
    rows = [tuple(int(x) for x in ln.split()) for ln in out.splitlines()]
    assert len(rows) == 2 * 9 * 9
    for overlap, op, k, rc, launches in rows:
        need = 2 if overlap and op == mspcg.OP_M5INV else FIELDS[op]
        if k < need:
            assert (rc, launches) == (mspcg.ENOMEM, 0), (overlap, op, k)
        else:
            assert rc == 0 and launches > 0, (overlap, op, k, rc)
