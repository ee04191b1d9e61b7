"""The wide-row GEMM's cache policies give the same bits.  A layer whose planes
start on a 128-byte line is loaded nontemporally past a size, the same layer 16
bytes further on is not; one and two token tiles, whole and ragged rows, dense
calls and experts on either side of the rows that count as one tile."""
import pytest
import torch

from gpu_helpers import DEV
from paper_2609_34380_amd import dps, workloads

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


def _shifted(nw):
    """The same layer, both planes 16 bytes off the line."""
    def move(t):
        buf = torch.empty(t.numel() + 16, dtype=torch.uint8, device=DEV)
        buf[16:].copy_(t.reshape(-1))
        return buf[16:]
    res = nw.residual
    return dps.NestedWeight(move(nw.hi).view(nw.hi.shape),
                            dps.Residual(move(res.pool), res.slots, res.log2_chunk), nw.enc)


def _layer(shape):
    w = torch.empty(shape, dtype=torch.float16, device=DEV)
    w.normal_(0.0, 0.02, generator=torch.Generator(device=DEV).manual_seed(4))
    return dps.split(w, dps.make_residual(w.numel(), 14, DEV))


def _same(a, b):
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("mode", [dps.MODE_FULL, dps.MODE_FAST], ids=["full", "fast"])
@pytest.mark.parametrize("m", [20, 40, 70, 200, 260])
def test_dense(m, mode):
    nw = _layer((10250, 8192))          # 80 MiB a plane, ragged last tile
    x = workloads.activations_fp16(m, 8192, seed=m).to(DEV)
    _same(dps.linear(x, nw, mode), dps.linear(x, _shifted(nw), mode))


@pytest.mark.parametrize("mode", [dps.MODE_FULL, dps.MODE_FAST], ids=["full", "fast"])
@pytest.mark.parametrize("n,k,rows", [(2048, 3072, 16 * 20), (2048, 3072, 16 * 40),
                                      (5136, 4096, 16 * 100), (5136, 4096, 16 * 150)])
def test_experts(n, k, rows, mode):
    experts = 16
    nw = _layer((experts, n, k))
    x = workloads.activations_fp16(rows, k, seed=2).to(DEV)
    cut = torch.randint(0, rows + 1, (experts - 1,), generator=torch.Generator().manual_seed(6))
    offsets = torch.cat([torch.zeros(1), cut.sort().values, torch.full((1,), rows)])
    offsets = offsets.to(torch.int32).to(DEV)
    _same(dps.linear_grouped(x, offsets, nw, mode),
          dps.linear_grouped(x, offsets, _shifted(nw), mode))
