"""Hop launches on both sides of the line between the small-launch kernel and the
general one (kernels.h, hop_is_small), every compiled Ls, against the FP64 oracle;
the FP16 matrix-core hop (hop_is_rows) against the FP64 operator.

Bars as in test_gpu_ops.py and test_gpu_mspcg.py: FP64 1e-13, FP32 1e-5, the block
operator in FP16 storage k16_bars()."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1804_08593_amd import mspcg, synth
from tests.gpu_util import cg16_bars, dev, host, k16_bars, relerr, say, setup, site_err

pytestmark = pytest.mark.gpu

# entries = sites per parity * Ls
SIZES = [
    ((8, 4, 6, 4), 2),      # small kernel, 32 sites a workgroup
    ((6, 4, 10, 2), 6),     # small, 60 of 64 lanes, ragged
    ((4, 6, 2, 8), 20),     # small, 3 sites a workgroup
    ((2, 6, 4, 4), 24),     # small, 2 sites
    ((4, 2, 6, 4), 32),     # small, 2 sites
    ((8, 8, 8, 10), 16),    # 40960 entries: small
    ((10, 14, 6, 18), 10),  # 75600 entries: general
    ((16, 12, 12, 20), 2),  # 46080 entries: general
    ((12, 12, 12, 14), 4),  # 48384 entries: general
    ((12, 10, 12, 10), 6),  # 43200 entries: general
    ((12, 12, 12, 12), 8),  # 82944 entries: general
    ((12, 10, 8, 10), 10),  # 48000 entries: general
    ((10, 6, 6, 12), 20),   # 43200 entries: general
    ((8, 8, 8, 8), 24),     # 49152 entries: general
    ((8, 8, 6, 8), 32),     # 49152 entries: general
]


@pytest.mark.parametrize("prec", [mspcg.FP64, mspcg.FP32])
@pytest.mark.parametrize("dims,Ls", SIZES, ids=lambda v: str(v))
def test_operators_across_launch_sizes(dims, Ls, prec):
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=31)
    psi = synth.fermion_field(dims, Ls, 32)
    e = O.parity_mask(act, psi, 0)
    d_in = dev(psi)
    tol = {mspcg.FP64: 1e-13, mspcg.FP32: 1e-5}[prec]
    for op, ref in ((mspcg.OP_HOP, O.hop(act, U, psi)), (mspcg.OP_D, O.dwf(act, U, psi)),
                    (mspcg.OP_DDAG, O.dwf(act, U, psi, dagger=True)),
                    (mspcg.OP_A, O.normal(act, U, e))):
        out = torch.zeros_like(d_in)
        ctx.apply(op, d_in, out, prec=prec)
        err = relerr(host(out), ref)
        say(f"{dims} Ls={Ls} prec={prec} op={op} relerr={err:.2e}")
        assert err <= tol, (op, err)


@pytest.mark.parametrize("dims,block,Ls", [
    ((8, 8, 4, 4), (4, 4, 4, 4), 8),      # every hop of the block operator small
    ((8, 8, 4, 4), (4, 4, 4, 4), 24),
    ((8, 8, 8, 4), (4, 4, 8, 4), 12),     # inner hops general, last hop small
    ((16, 8, 8, 8), (8, 8, 8, 8), 16),    # every hop general
    ((16, 8, 8, 8), (8, 8, 8, 8), 20),
], ids=lambda v: str(v))
@pytest.mark.parametrize("prec", [mspcg.FP64, mspcg.FP32, mspcg.FP16])
def test_block_operator_across_launch_sizes(dims, block, Ls, prec):
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=33)
    p = O.parity_mask(act, synth.fermion_field(dims, Ls, 34), 0)
    ctx.set_blocking(block, 2)
    out = torch.zeros_like(dev(p))
    ctx.apply(mspcg.OP_KBLOCK, dev(p), out, prec=prec)
    ref = O.block_precond_op(act, U, p, block, "literal")
    err, se = relerr(host(out), ref), site_err(host(out), ref)
    n16, s16 = k16_bars()
    bar = {mspcg.FP64: (1e-13, 1e-12), mspcg.FP32: (1e-5, 1e-4), mspcg.FP16: (n16, s16)}[prec]
    say(f"K {dims} {block} Ls={Ls} prec={prec}: {err:.2e} per entry {se:.2e}")
    assert err <= bar[0] and se <= bar[1]


@pytest.mark.parametrize("dims,block,pad,c", [
    ((24, 24, 24, 24), (24, 24, 12, 24), 2, 0.5),  # one cut direction, the others periodic
    ((20, 28, 18, 32), (10, 14, 6, 16), 2, 0.5),   # odd half extents in every direction
    ((20, 28, 18, 32), (20, 14, 18, 16), 1, 0.5),  # periodic x and z, pad 1
    ((16, 24, 28, 32), (8, 12, 14, 16), 0, 0.5),   # no pad
    ((16, 24, 28, 32), (4, 12, 14, 16), 2, 0.0),   # Shamir, blocks as short as a piece in x
], ids=lambda v: str(v))
def test_matrix_core_hop(dims, block, pad, c):
    Ls, l = 16, 2
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.0 + c, c, gseed=35)
    gen = torch.Generator(device="cuda").manual_seed(36)
    p = torch.randn(ctx.fshape, dtype=torch.complex128, device="cuda", generator=gen)
    ctx.set_blocking(block, pad)
    ref, out = torch.zeros_like(p), torch.zeros_like(p)
    for run, bars in ((lambda o, prec: ctx.apply(mspcg.OP_KBLOCK, p, o, prec=prec), k16_bars()),
                      (lambda o, prec: ctx.precond(p, o, l, prec=prec), cg16_bars(l))):
        run(ref, mspcg.FP64)
        run(out, mspcg.FP16)
        err, se = relerr(host(out), host(ref)), site_err(host(out), host(ref))
        say(f"{dims} {block} pad={pad} c={c}: {err:.2e} per entry {se:.2e}")
        assert err <= bars[0] and se <= bars[1]


@pytest.mark.parametrize("prec", [mspcg.FP64, mspcg.FP32, mspcg.FP16])
@pytest.mark.parametrize("dims,block,Ls", [
    ((6, 4, 6, 4), (2, 4, 2, 4), 2),     # a workgroup holds more sites than a block
    ((8, 6, 6, 4), (4, 2, 6, 4), 6),     # 60 of 64 lanes, a ragged last workgroup
    ((6, 8, 4, 8), (6, 4, 4, 2), 20),
    ((4, 6, 8, 4), (4, 6, 4, 4), 32),
], ids=lambda v: str(v))
def test_preconditioner_fields_in_and_out(dims, block, Ls, prec):
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=37)
    r = synth.fermion_field(dims, Ls, 38)  # odd sites are ignored
    ctx.set_blocking(block, 2)
    z = torch.full_like(dev(r), 7.0)
    for l in (0, 1):
        ctx.precond(dev(r), z, l, prec=prec)
        got = host(z)
        assert np.all(O.parity_mask(act, got, 1) == 0)
        ref = O.inner_block_cg(act, U, O.parity_mask(act, r, 0), block, l, "literal")
        bar = {mspcg.FP64: (1e-12, 1e-11), mspcg.FP32: (1e-5, 1e-4), mspcg.FP16: cg16_bars(l)}[prec]
        err, se = relerr(got, ref), site_err(got, ref)
        say(f"precond {dims} {block} Ls={Ls} prec={prec} l={l}: {err:.2e} per entry {se:.2e}")
        assert err <= bar[0] and se <= bar[1]
