"""Per-length transforms while other streams keep the chip busy: the waves of a
block then run apart, and a wave that reads a tile before another one's last
LDS writes have arrived gives other bits.  Each stage and the whole solve give
the bits of the same call alone; lengths whose last round of placement is
ragged (108 = 2 * 54 over 16 lines), along x and along y, types IV and others."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    ((108, 192, 100), ("DN", "NN", "NN")),
    ((108, 90, 150), ("NN", "ND", "DD")),
    ((180, 108, 100), ("P", "DD", "NN")),
]


@pytest.mark.parametrize("shape,bcs", CASES)
def test_same_bits_beside_other_streams(shape, bcs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import Plan

    def plan(nx, ny, nz, b):
        return Plan(nx, ny, nz, 1.0 / nx, 1.0 / ny, np.full(nz, 1.0 / nz), b)

    p = plan(*shape, bcs)
    others = [((180, 300, 96), ("ND", "NN", "NN")), ((216, 192, 72), ("DN", "ND", "P"))]
    busy = [(plan(*s, b), torch.zeros(s[::-1], device="cuda", dtype=torch.float64), torch.cuda.Stream())
            for s, b in others]
    stream = torch.cuda.Stream()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(shape))
    f = torch.rand(shape[::-1], generator=gen, device="cuda", dtype=torch.float64)
    ops = {f"transform {role} {'inverse' if inv else 'forward'}":
           (lambda x, role=role, inv=inv: p.transform_stage(role, inv, x, stream=stream))
           for role in (0, 1) for inv in (False, True)}
    ops["elimination"] = lambda x: p.tridiag_stage(x, stream=stream)
    ops["solve"] = lambda x: p.solve(x, stream=stream)
    for name, op in ops.items():
        alone = f.clone()
        torch.cuda.synchronize()
        op(alone)
        torch.cuda.synchronize()
        for rep in range(15):
            print("streams", shape, bcs, name, rep, flush=True)
            fields = [f.clone() for _ in range(6)]
            torch.cuda.synchronize()
            for x in fields:
                for q, g, s in busy:
                    q.solve(g, stream=s)
                op(x)
            torch.cuda.synchronize()
            assert all(torch.equal(x, alone) for x in fields), (name, rep)
