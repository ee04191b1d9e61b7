"""The 256 x 256 FP16 tile's residual pointers: a wave keeps one pointer per
line and renews them where a line leaves its residual chunk or passes the end
of the K range, walking K forwards or backwards (odd groups of four weight
tiles).  Chunks from 16 bytes (every piece its own chunk) to longer than a
row, on a K range that ends inside a stage, against the oracle; and table
entries outside the pool, which read as zero residual bytes, bit for bit
against the same layer with those chunks zeroed."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, Nested, assert_close, u16
from paper_2609_34380_amd import dps, workloads

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]

M, N, K = 1800, 8456, 464      # 8 x 34 tiles: whole groups both ways, ragged edges


def _layer(log2c, enc=dps.ENC_E5M2):
    n_chunks = -(-N * K // (1 << log2c))
    return Nested(workloads.weight_fp16(N, K, seed=77), log2c, n_slots=n_chunks + 9,
                  slot_seed=log2c, filler_seed=5, enc=enc)


@pytest.mark.parametrize("log2c,enc", [(4, dps.ENC_E5M2), (5, dps.ENC_E4M3), (6, dps.ENC_E5M2),
                                       (8, dps.ENC_E4M3), (11, dps.ENC_E5M2)])
def test_chunks_of_any_size(log2c, enc):
    p = dps.plan_info(dps.MODE_FULL, "fp16", M, N, K, log2_chunk=log2c)
    assert (p["tile_rows"], p["tile_tokens"], p["splits"]) == (256, 256, 1)
    nst = _layer(log2c, enc)
    x = workloads.activations_fp16(M, K, seed=78)
    y = dps.linear(x.to(DEV), nst.nw, dps.MODE_FULL)
    rows = np.concatenate([np.arange(0, 256, 16), np.arange(M - 8, M)])
    ref = oracle.linear_rows(oracle.FULL, u16(x), rows, nst.hi_ref, nst.res_ref, enc=enc)
    assert_close(y[torch.from_numpy(rows).to(DEV)], ref, "log2c=%d" % log2c)


@pytest.mark.parametrize("log2c", [6, 11])
def test_slots_outside_the_pool_read_as_zero(log2c):
    nst = _layer(log2c)
    x = workloads.activations_fp16(M, K, seed=79).to(DEV)
    slots = nst.res.slots.clone()
    lost = torch.arange(1, slots.numel(), 7, device=DEV)
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


@pytest.mark.parametrize("m,n,k,splits", [
    (700, 16650, 464, 1),     # 198 tiles, ragged every way
    (700, 8190, 8208, 2),     # 96 tiles in two K ranges, N not a multiple of 4
])
@pytest.mark.parametrize("mode", [dps.MODE_FAST, dps.MODE_FULL], ids=["fast", "full"])
def test_part_filled_grids_take_the_tile(m, n, k, splits, mode):
    p = dps.plan_info(mode, "fp16", m, n, k)
    assert (p["tile_rows"], p["tile_tokens"], p["splits"]) == (256, 256, splits)
    nst = Nested(workloads.weight_fp16(n, k, seed=81), 14, slot_seed=3)
    x = workloads.activations_fp16(m, k, seed=82)
    y = dps.linear(x.to(DEV), nst.nw, mode)
    rows = np.concatenate([np.arange(0, m, 37), [m - 1]])
    ref = oracle.linear_rows(oracle.FAST if mode == dps.MODE_FAST else oracle.FULL, u16(x), rows,
                             nst.hi_ref, nst.res_ref if mode == dps.MODE_FULL else None)
    assert_close(y[torch.from_numpy(rows).to(DEV)], ref)


def test_small_workspace_still_runs():
    """A call whose K ranges need a workspace runs with a smaller one, on the
    128-row tile; a call that cannot do without stays refused."""
    m, n, k = 700, 8190, 8208
    ws = torch.empty(256, dtype=torch.uint8, device=DEV)
    assert dps.workspace_bytes(dps.MODE_FAST, dps.ACT_FP16, m, n, k, 1) > ws.numel()
    nst = Nested(workloads.weight_fp16(n, k, seed=83), 14, slot_seed=3)
    x = workloads.activations_fp16(m, k, seed=84)
    y = dps.linear(x.to(DEV), nst.nw, dps.MODE_FAST, workspace=ws)
    rows = np.concatenate([np.arange(0, m, 37), [m - 1]])
    ref = oracle.linear_rows(oracle.FAST, u16(x), rows, nst.hi_ref, None)
    assert_close(y[torch.from_numpy(rows).to(DEV)], ref)
    assert dps.workspace_bytes(dps.MODE_FAST, dps.ACT_FP16, 40, n, k, 1) > ws.numel()
    with pytest.raises(dps.DpsError):
        dps.linear(x[:40].contiguous().to(DEV), nst.nw, dps.MODE_FAST, workspace=ws)


def test_misaligned_workspace_still_runs():
    """So does one off its alignment, in a call that the 128-row tile serves
    without any; where that tile needs one too, it is refused."""
    m, n, k = 1300, 4096, 4096
    assert dps.plan_info(dps.MODE_FAST, "fp16", m, n, k)["splits"] == 2
    need = dps.workspace_bytes(dps.MODE_FAST, dps.ACT_FP16, m, n, k, 1)
    ws = torch.empty(need + 16, dtype=torch.uint8, device=DEV)[16:]
    nst = Nested(workloads.weight_fp16(n, k, seed=85), 14, slot_seed=3)
    x = workloads.activations_fp16(m, k, seed=86)
    y = dps.linear(x.to(DEV), nst.nw, dps.MODE_FAST, workspace=ws)
    rows = np.concatenate([np.arange(0, m, 67), [m - 1]])
    ref = oracle.linear_rows(oracle.FAST, u16(x), rows, nst.hi_ref, None)
    assert_close(y[torch.from_numpy(rows).to(DEV)], ref)
    with pytest.raises(dps.DpsError):
        dps.linear(x[:40].contiguous().to(DEV), nst.nw, dps.MODE_FAST, workspace=ws)
