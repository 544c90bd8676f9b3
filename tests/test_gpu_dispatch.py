"""The general hop kernel where launches are too large for the small-launch one: its
traversal tiles and its writes of boundary fields; local solves whose hops take
different kernels; the FP16 matrix-core hop on the split form and on uncut lattices.

Bars as in test_gpu_ops.py and test_gpu_mspcg.py: FP64 1e-13, FP32 1e-5, FP16 storage
k16_bars() and cg16_bars(l)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1804_08593_amd import mspcg, synth
from tests.gpu_util import cg16_bars, dev, host, k16_bars, relerr, say, setup, site_err
from tests.test_gpu_ops import OPS, _ref

pytestmark = pytest.mark.gpu

SMALL_MOST = 42000  # entries (sites * Ls over all blocks) of the largest small launch
EVEN_OUT = (mspcg.OP_MHAT, mspcg.OP_MHATDAG, mspcg.OP_A, mspcg.OP_PREPARE)


def entries(dims, Ls):
    return int(np.prod(dims)) // 2 * Ls


@pytest.mark.parametrize("tile", [
    (1 << 16, 4, 8, 16),   # whole rows, clamped in x (and in y, z, t where it must)
    (8, 4, 4, 4), (2, 2, 2, 2), (6, 14, 6, 20),
    (1 << 16, 1 << 16, 1 << 16, 1 << 16),  # one tile
], ids=str)
@pytest.mark.parametrize("dims,Ls,blk", [
    ((16, 12, 12, 20), 8, (8, 12, 6, 10)),
    ((10, 14, 18, 12), 6, (10, 14, 6, 6)),
], ids=lambda v: str(v))
def test_tiles_of_the_general_hop_are_bitwise_identical(dims, Ls, blk, tile):
    """Whole-lattice hops, and with pad 0 every hop of the block operator, visit their
    sites in the order of the tile here: same bits as in lexicographic order."""
    assert entries(dims, Ls) > SMALL_MOST  # the blocks' interiors together hold as many
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=51)
    psi = synth.fermion_field(dims, Ls, 52)
    d = dev(psi)
    runs = [(f"op {op} prec {prec}", (lambda o, op=op, prec=prec: ctx.apply(op, d, o, prec=prec)))
            for op in (mspcg.OP_A, mspcg.OP_D) for prec in (mspcg.FP64, mspcg.FP32)]
    for pad in (0, 2):
        for prec in (mspcg.FP64, mspcg.FP32, mspcg.FP16):
            def k(o, pad=pad, prec=prec):
                ctx.set_blocking(blk, pad)
                ctx.apply(mspcg.OP_KBLOCK, d, o, prec=prec)

            def pc(o, pad=pad, prec=prec):  # the hop with the fused update too
                ctx.set_blocking(blk, pad)
                ctx.precond(d, o, 2, prec=prec)
            runs += [(f"K pad {pad} prec {prec}", k), (f"precond pad {pad} prec {prec}", pc)]
    for name, run in runs:
        ref, out = torch.full_like(d, float("nan")), torch.full_like(d, float("nan"))
        ctx.set_tuning(1, (0, 0, 0, 0), (0, 0, 0, 0), (0, 0, 0, 0))
        run(ref)
        for remap in (0, 1):
            say(f"{dims} Ls={Ls} tile {tile} remap {remap}: {name}")
            ctx.set_tuning(remap, tile, tile, tile)
            run(out)
            if "precond" in name:
                # sums over a block's workgroups in another order: the step lengths may
                # differ in the last bits, the fields by the storage's unit
                unit = {0: 1e-13, 1: 1e-6, 2: 2.0 ** -11}[int(name[-1])]
                assert relerr(host(out), host(ref)) <= unit
            else:
                assert torch.equal(out, ref)
    e = O.parity_mask(act, psi, 0)
    out = torch.full_like(d, float("nan"))
    ctx.apply(mspcg.OP_A, d, out)
    assert relerr(host(out), O.normal(act, U, e)) <= 1e-13


GENERAL = [
    ((16, 12, 12, 20), 2),  # full workgroups
    ((12, 10, 12, 10), 6),  # 252 of 256 threads, a ragged last workgroup
    ((10, 14, 6, 18), 10),  # 250 threads, ragged
    ((10, 6, 6, 12), 20),   # 240 threads, ragged
    ((8, 8, 10, 6), 24),    # 240 threads
    ((8, 8, 6, 8), 32),
    ((8, 8, 10, 10), 16),
]


@pytest.mark.parametrize("prec", [mspcg.FP64, mspcg.FP32])
@pytest.mark.parametrize("dims,Ls", GENERAL, ids=lambda v: str(v))
def test_boundary_fields_written_by_the_general_hop(dims, Ls, prec):
    """Every operator into a field of NaN: all sites written, the odd ones of even
    results with zeros."""
    assert entries(dims, Ls) > SMALL_MOST
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=53)
    psi = synth.fermion_field(dims, Ls, 54)
    d_in = dev(psi)
    for op in OPS:
        out = torch.full_like(d_in, float("nan"))
        ctx.apply(op, d_in, out, prec=prec)
        got = host(out)
        assert np.isfinite(got).all(), op
        err = relerr(got, _ref(op, act, U, psi))
        say(f"{dims} Ls={Ls} prec={prec} op={op} relerr={err:.2e}")
        assert err <= {mspcg.FP64: 1e-13, mspcg.FP32: 1e-5}[prec], (op, err)
        if op in EVEN_OUT:
            assert np.all(O.parity_mask(act, got, 1) == 0)


@pytest.mark.parametrize("dims,block,Ls", [
    ((16, 12, 12, 20), (16, 12, 6, 10), 2),  # links loaded by every thread, not staged
    ((16, 12, 12, 10), (8, 12, 12, 10), 4),
    ((12, 10, 12, 10), (6, 10, 12, 10), 6),
    ((8, 8, 10, 6), (4, 8, 10, 6), 24),
    ((8, 8, 6, 8), (8, 8, 6, 4), 32),
], ids=lambda v: str(v))
def test_fp16_block_operator_on_the_general_hop(dims, block, Ls):
    assert entries(dims, Ls) > SMALL_MOST
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=61)
    p = O.parity_mask(act, synth.fermion_field(dims, Ls, 62), 0)
    for pad, mode in ((0, "dirichlet"), (2, "literal")):
        ctx.set_blocking(block, pad)
        out = torch.full_like(dev(p), float("nan"))
        ctx.apply(mspcg.OP_KBLOCK, dev(p), out, prec=mspcg.FP16)
        ref = O.block_precond_op(act, U, p, block, mode)
        err, se = relerr(host(out), ref), site_err(host(out), ref)
        say(f"K {dims} {block} pad={pad} Ls={Ls}: {err:.2e} per entry {se:.2e}")
        assert err <= k16_bars()[0] and se <= k16_bars()[1]


@pytest.mark.parametrize("prec", [mspcg.FP64, mspcg.FP32, mspcg.FP16])
@pytest.mark.parametrize("dims,block,pad,Ls", [
    # u onto 82944 entries general, the last hop onto 16384 small
    ((8, 8, 8, 8), (4, 4, 4, 4), 2, 8),
    # 640 workgroups a hop: small, but for the FP16 hop with the fused update
    ((8, 8, 8, 20), (8, 8, 8, 10), 0, 8),
    # u and v 768 workgroups, last hop 512: FP64 general and small, FP32 and FP16 small
    ((4, 8, 8, 8), (4, 8, 8, 4), 2, 24),
], ids=lambda v: str(v))
def test_local_solve_with_hops_on_different_kernels(dims, block, pad, Ls, prec):
    """The two reductions of a step then count the workgroups of different kernels."""
    l = 3
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=55)
    r = synth.fermion_field(dims, Ls, 56)
    ctx.set_blocking(block, pad)
    z = torch.full_like(dev(r), float("nan"))
    ctx.precond(dev(r), z, l, prec=prec)
    ref = O.inner_block_cg(act, U, O.parity_mask(act, r, 0), block, l,
                           "dirichlet" if pad == 0 else "literal")
    bar = {mspcg.FP64: (1e-12, 1e-11), mspcg.FP32: (1e-5, 1e-4), mspcg.FP16: cg16_bars(l)}[prec]
    err, se = relerr(host(z), ref), site_err(host(z), ref)
    say(f"precond {dims} {block} pad={pad} Ls={Ls} prec={prec}: {err:.2e} per entry {se:.2e}")
    assert err <= bar[0] and se <= bar[1]


@pytest.mark.parametrize("dims,block,pad,form", [
    ((24, 24, 24, 24), (24, 24, 12, 24), 2, mspcg.FORM_SPLIT),  # y hop onto the block alone
    ((20, 28, 18, 32), (10, 14, 18, 16), 1, mspcg.FORM_SPLIT),
    ((24, 24, 24, 24), (24, 24, 24, 24), 2, mspcg.FORM_DOMAIN),  # every direction periodic
    ((18, 26, 28, 24), (18, 26, 28, 24), 0, mspcg.FORM_DOMAIN),  # odd half extents
], ids=lambda v: str(v))
def test_matrix_core_hop_split_form_and_uncut_lattices(dims, block, pad, form):
    Ls, l = 16, 2
    assert int(np.prod(dims)) // 2 >= 150000  # the launches of the matrix-core hop
    act, U, ctx = setup(dims, Ls, 1.8, 0.05, 1.5, 0.5, gseed=57)
    p = torch.randn(ctx.fshape, dtype=torch.complex128, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(58))
    ctx.set_blocking(block, pad, form)
    ref, out = torch.full_like(p, float("nan")), torch.full_like(p, float("nan"))
    for run, bars in ((lambda o, prec: ctx.apply(mspcg.OP_KBLOCK, p, o, prec=prec), k16_bars()),
                      (lambda o, prec: ctx.precond(p, o, l, prec=prec), cg16_bars(l))):
        run(ref, mspcg.FP64)
        run(out, mspcg.FP16)
        err, se = relerr(host(out), host(ref)), site_err(host(out), host(ref))
        say(f"{dims} {block} pad={pad} form={form}: {err:.2e} per entry {se:.2e}")
        assert err <= bars[0] and se <= bars[1]
