"""The wide-row GEMM's residual pointers.  A wave that loads residual bytes
keeps one pointer per piece: the rows of a K range no longer than a chunk have
two chunks at most, whose slots are read once, and a piece changes over at the
stage where its row does; shorter chunks are looked up stage by stage.  Walks
start at stage 0, or (K a multiple of 4096) at another stage for every group of
four weight tiles and wrap.  K ranges that end inside a stage, 32-, 64- and
128-token tiles and experts, against the oracle; and table entries outside the
pool, which read as zero residual bytes, bit for bit against the same layer
with those chunks zeroed."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, Nested, assert_close, u16
from paper_2609_34380_amd import dps, workloads

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

LAYERS = [
    # n, k, log2c: where a row crosses chunks
    (2100, 784, 14),    # one row in 20 crosses, K ends 16 elements into a stage
    (1152, 1040, 10),   # chunks shorter than a row, off its grid
    (2052, 4112, 16),   # two K ranges and more, crossings in both
    (1300, 12288, 14),  # rotated walk, three of four rows cross
    (1300, 4096, 9),    # rotated walk, eight chunks a row
    (1300, 8192, 11),   # rotated walk, a chunk every sixteen stages
    (700, 144, 4),      # every piece its own chunk
]


@pytest.mark.parametrize("m", [24, 60, 150])
@pytest.mark.parametrize("enc", [dps.ENC_E5M2, dps.ENC_E4M3], ids=["e5m2", "e4m3"])
@pytest.mark.parametrize("n,k,log2c", LAYERS)
def test_rows_across_chunks(n, k, log2c, enc, m):
    p = dps.plan_info(dps.MODE_FULL, "fp16", m, n, k, log2_chunk=log2c)
    assert p["tile_rows"] == 128
    chunks = -(-n * k // (1 << log2c))
    nst = Nested(workloads.weight_fp16(n, k, seed=n), log2c, n_slots=chunks + 5, slot_seed=m,
                 filler_seed=6, enc=enc)
    x = workloads.activations_fp16(m, k, seed=m)
    y = dps.linear(x.to(DEV), nst.nw, dps.MODE_FULL)
    rows = np.unique(np.concatenate([np.arange(0, m, 11), [m - 1]]))
    ref = oracle.linear_rows(oracle.FULL, u16(x), rows, nst.hi_ref, nst.res_ref, enc=enc)
    assert_close(y[torch.from_numpy(rows).to(DEV)], ref)


@pytest.mark.parametrize("rows", [100, 700])
def test_experts_across_chunks(rows):
    experts, n, k, log2c = 5, 520, 1552, 14
    w = workloads.weight_fp16(experts * n, k, seed=3).reshape(experts, n, k)
    nst = Nested(w, log2c, slot_seed=7)
    x = workloads.activations_fp16(rows, k, seed=8)
    offsets = np.array([0, rows // 5, rows // 5, rows // 2, rows - 3, rows], np.int32)
    y = dps.linear_grouped(x.to(DEV), torch.from_numpy(offsets).to(DEV), nst.nw, dps.MODE_FULL)
    assert_close(y, oracle.linear_grouped(oracle.FULL, u16(x), offsets, nst.hi_ref, nst.res_ref))


@pytest.mark.parametrize("n,k,log2c", [(2100, 784, 14), (1300, 12288, 14), (1300, 4096, 9)])
def test_slots_outside_the_pool_read_as_zero(n, k, log2c):
    nst = Nested(workloads.weight_fp16(n, k, seed=5), log2c, slot_seed=1, filler_seed=5)
    x = workloads.activations_fp16(40, k, seed=9).to(DEV)
    slots = nst.res.slots.clone()
    lost = torch.arange(1, slots.numel(), 5, device=DEV)
    pool = nst.res.pool.clone()
    pool.view(-1, 1 << log2c)[slots[lost].long()] = 0
    want = dps.linear(x, dps.NestedWeight(nst.nw.hi, dps.Residual(pool, slots, log2c)),
                      dps.MODE_FULL)
    bad = slots.clone()
    bad[lost[::2]] = -1
    bad[lost[1::2]] = pool.numel() >> log2c
    got = dps.linear(x, dps.NestedWeight(nst.nw.hi, dps.Residual(nst.res.pool, bad, log2c)),
                     dps.MODE_FULL)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
