"""Transfers and reductions at the edges of their units of four cells: fields of
fewer than four cells, rows that end inside a unit, sources and destinations at
every alignment a cell has. Transferred values are exact; a reduction's are those
of FP64 sums to the rounding of n additions, n 2^-53 of the sum of magnitudes
(each side)."""
import numpy as np
import pytest

from paper_1004_0480_amd import rd
from paper_1004_0480_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 1, 3), (3, 1, 1), (2, 2, 2), (3, 5, 7), (2, 3, 64), (5, 9, 130), (300, 3, 1), (9, 7, 403), (2, 3, 4096)]


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
def test_transfers_and_reductions_at_unit_edges(storage):
    import torch
    kind = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[storage]
    gen = torch.Generator().manual_seed(4)
    for shape in SHAPES:
        n = int(np.prod(shape))
        flat = torch.rand(n + 3, generator=gen, dtype=torch.float64) * 5.0 - 2.0
        g = rd.Grid(shape, 1, 0.5, storage)
        g.set_model(W.ModelSpec("diffusion", 1, 0.01, 0.5, [[1.0] * 3], W.uniform_bc(1, "mirror")))
        for shift in range(4):
            for src in (torch.float64, torch.float32, torch.bfloat16, torch.float16):
                x = flat.to(src).cuda()[shift:shift + n].view(shape)
                want = x.float().to(kind).double()
                g.write(0, x)
                out = torch.full((n + 8,), 7.0, device="cuda")
                dst = out[shift:shift + n].view(shape)
                g.read_device(0, dst)
                assert torch.equal(dst.double(), want), (shape, shift, src)
                assert bool((out[:shift] == 7.0).all()) and bool((out[shift + n:] == 7.0).all())
                assert np.array_equal(g.read(0), want.cpu().numpy())
                w = want.cpu().numpy().ravel()
                res = torch.zeros(2, dtype=torch.float64, device="cuda")
                sums = [g.reduce(0)]
                if src == kind:
                    rd.reduce_noalloc(x.data_ptr(), storage, shape, 0.5, res.data_ptr())
                    torch.cuda.synchronize()
                    sums.append(tuple(res.tolist()))
                for got in sums:
                    for s, terms in zip(got, (w, w * w)):
                        tol = 2.0 * (n + 4) * 2.0 ** -53 * np.abs(terms).sum() * 0.125
                        assert abs(s - terms.sum() * 0.125) <= tol, (shape, shift, src)
        g.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_rows_longer_than_a_workgroup_takes(storage):
    """Long rows are split between workgroups: rows that end inside a part's
    last unit, one row and several, every value exact."""
    import torch
    for shape in ((1, 1, 70001), (1, 3, 5003), (2, 2, 16384), (1, 1, 1 << 20)):
        x = (torch.arange(int(np.prod(shape))) % 251).float().cuda().view(shape)    # exact in BF16
        g = rd.Grid(shape, 1, 1.0, storage)
        g.set_model(W.ModelSpec("diffusion", 1, 0.01, 1.0, [[1.0] * 3], W.uniform_bc(1, "mirror")))
        g.write(0, x)
        out = torch.full(shape, -1.0, device="cuda")
        g.read_device(0, out)
        assert torch.equal(out, x), shape
        assert np.array_equal(g.read(0), x.double().cpu().numpy())
        g.close()
