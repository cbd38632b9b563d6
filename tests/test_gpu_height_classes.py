"""Batches of every height class, and the direct kernel at every alignment an
element may have (GPU): all storage types, against pw_advect bit for bit and
against the oracle within the arithmetic bound of the type."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, max_rel, say
from paper_2107_13500_amd import batched as BT
from paper_2107_13500_amd import binding as B
from paper_2107_13500_amd import inputs, metrics
from test_gpu_precision import arith_bound

pytestmark = pytest.mark.gpu

STORAGES = [B.F64, B.F32, B.BF16, B.F16, B.I16, B.I32]
IDS = ["f64", "f32", "bf16", "f16", "i16", "i32"]


def same_bytes(a, b):
    return torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


def bound_of(storage, out_scale, ref):
    m = float(np.max(np.abs(ref)))
    if storage == B.F64:
        return metrics.F64_PARITY_TOL
    return arith_bound(storage, out_scale, m) if m > 0 else 0.0


@pytest.mark.parametrize("storage", STORAGES, ids=IDS)
@pytest.mark.parametrize("chunk", [256, 512, 1024])
@pytest.mark.parametrize("heights", [(84, 2, 40), (83, 3, 84), (86, 4, 170), (85, 5, 170), (172, 6, 256), (171, 7, 255)],
                         ids=["even84", "any84", "even170", "any170", "even256", "any256"])
def test_batches_of_every_height_class(storage, chunk, heights):
    """A batch runs the kernel of its tallest column's class, even heights or
    any: columns at the class's edges, one far shorter than the class, chunks
    that end after one point (171 rows of height 3, 25 of 41, 27 of 19)."""
    lo, short, hi = heights
    shapes = [(7, 13, lo), (5, 4, short), (3, 5, hi), (2, 1, lo), (11, 2, hi), (4, 171, short)]
    if hi == 84 and lo % 2:
        shapes += [(3, 171, 3), (4, 25, 41), (2, 27, 19)]
    probs = [inputs.make_problem(*s, seed=8000 + d) for d, s in enumerate(shapes)]
    say("height class", B.DTYPE_NAMES[storage], chunk, heights)
    batch = BT.DeviceBatch(probs, storage, DEV)
    tuning = {"chunk": chunk, "seg": 4}
    plan = batch.plan(tuning)
    batch.advect(plan)
    torch.cuda.synchronize()
    assert plan.error_count() == 0
    got = [[o.clone() for o in f[3:]] for f in batch.fields]
    skipped = torch.zeros(1, dtype=torch.int64, device=DEV)
    for d, (f, p, sc) in enumerate(zip(batch.fields, probs, batch.scales)):
        outs = [torch.zeros_like(f[0]) for _ in range(3)]
        single = B.Plan(storage, [batch.shapes[d]], dict(tuning, variant=B.VARIANT_MARCH))
        B.advect(single, *f[:3], *outs, p.coeffs.tcx, p.coeffs.tcy, *batch.tz[d],
                 scales=sc if storage in B.SCALED else None)
        torch.cuda.synchronize()
        for a, b in zip(got[d], outs):
            assert same_bytes(a, b), "domain %d differs from pw_advect" % d
        ref = oracle.advect(*batch.host_fields(d), p.coeffs.tcx, p.coeffs.tcy, *p.coeffs.arrays())
        for q, (g, r) in enumerate(zip(batch.host_outputs(d), ref)):
            r = r[1:-1, 1:-1]
            assert max_rel(g[1:-1, 1:-1], r) <= bound_of(storage, float(sc.out_scale[q]), r), (d, q)
    for default in (False, True):   # without a plan; default segments too
        for f in batch.fields:
            for o in f[3:]:
                o.zero_()
        B.advect_batched_noalloc(storage, batch.shapes, batch.d_args, {"chunk": chunk} if default else tuning, skipped)
        torch.cuda.synchronize()
        assert int(skipped.item()) == 0
        for d, f in enumerate(batch.fields):
            for a, b in zip(got[d], f[3:]):
                assert same_bytes(a, b), "without a plan: domain %d differs" % d


@pytest.mark.parametrize("storage", STORAGES, ids=IDS)
@pytest.mark.parametrize("shape,pad,plane,shift", [((9, 4, 30), 1, 0, 0), ((6, 3, 124), 3, 1, 1), ((5, 5, 2), 1, 0, 1),
                                                   ((7, 3, 62), 0, 1, 0), ((4, 62, 64), 0, 0, 1), ((4, 3, 31), 0, 0, 0),
                                                   ((3, 5, 63), 0, 0, 1), ((3, 1, 257), 2, 1, 1)],
                         ids=lambda s: str(s).replace(", ", "x"))
def test_direct_kernel_at_every_element_alignment(storage, shape, pad, plane, shift):
    """Pairs of levels at odd elements: even heights with an odd column pitch,
    an odd plane stride or bases one element off, and odd planes, whose last
    pair ends with the plane.  The buffer accesses of a pair are then aligned to
    one element only (2 bytes for the 16-bit types): every value within the
    bound, nothing written outside the interior columns."""
    nx, ny, nz = shape
    p = inputs.make_problem(*shape, seed=8100 + nx + ny + nz)
    ins, outs = inputs.storage_scales(p, B.DTYPE_NAMES[storage])
    sy = nz + pad
    sx = (ny + 2) * sy + plane
    size = (nx + 1) * sx + (ny + 1) * sy + nz
    bufs = [torch.full((size + shift,), -77, dtype=B.torch_dtype(storage), device=DEV) for _ in range(6)]
    v = [b[shift:].as_strided((nx + 2, ny + 2, nz), (sx, sy, 1)) for b in bufs]
    for t, a, s in zip(v, (p.u, p.v, p.w), ins):
        t.copy_(B.to_storage(a, storage, s, DEV))
    c = p.coeffs
    tz = [torch.from_numpy(x).to(DEV) for x in c.arrays()]
    say("direct alignment", B.DTYPE_NAMES[storage], shape, pad, plane, shift)
    plan = B.Plan(storage, [B.shape_of(v[0])], {"variant": B.VARIANT_DIRECT})
    B.advect(plan, *v, c.tcx, c.tcy, *tz, scales=B.make_scales(ins, outs))
    torch.cuda.synchronize()
    deq = [np.ascontiguousarray(B.from_storage(t, storage, s)) for t, s in zip(v[:3], ins)]
    ref = oracle.advect(*deq, c.tcx, c.tcy, *c.arrays())
    for t, r, s in zip(v[3:], ref, outs):
        g, r = B.from_storage(t, storage, s)[1:-1, 1:-1], r[1:-1, 1:-1]
        assert max_rel(g, r) <= bound_of(storage, s, r)
        t[1:-1, 1:-1] = -77
    assert all(bool((b == -77).all()) for b in bufs[3:]), "written outside the interior columns"
