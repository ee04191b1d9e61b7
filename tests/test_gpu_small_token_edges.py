"""Edges of the small-token kernels and of the encoding choice.

The 16-row kernel stages eight token rows up to eight tokens and sixteen
beyond; the row GEMV takes one weight row per wave for one token in full mode
beyond 8192 rows of 1536 elements on, two below.  Both against the oracle on ragged K and row counts.  The
encoding choice reads four vectors per thread: a misfit in any vector of a
layer that ends inside a block's share flips it."""
import pytest
import torch

import oracle
from gpu_helpers import DEV, Nested, assert_close, u16
from paper_2609_34380_amd import dps, workloads

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

MODES = {"fast": (dps.MODE_FAST, oracle.FAST), "full": (dps.MODE_FULL, oracle.FULL)}


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("m", [5, 8, 9])
@pytest.mark.parametrize("n,k,log2c,enc", [
    (4085, 1040, 12, dps.ENC_E5M2),   # one row group per block, ragged rows, 16-element K tail
    (4112, 5136, 9, dps.ENC_E4M3),    # two groups, chunks below 1 KiB
])
def test_token_rows_staged(n, k, log2c, enc, m, mode):
    dmode, omode = MODES[mode]
    nst = Nested(workloads.weight_fp16(n, k, seed=n), log2c, slot_seed=m, enc=enc)
    x = workloads.activations_fp16(m, k, seed=m)
    ref = oracle.linear(omode, u16(x), nst.hi_ref, nst.res_ref if mode == "full" else None,
                        enc=enc)
    assert_close(dps.linear(x.to(DEV), nst.nw, dmode), ref)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n,k,log2c,enc", [
    (8193, 1040, 10, dps.ENC_E5M2),   # just past the two-row rule, a part-filled last block
    (8203, 1536, 14, dps.ENC_E5M2),   # the shortest rows taken one by one, and just below
    (8203, 1520, 14, dps.ENC_E4M3),
    (8203, 2064, 14, dps.ENC_E4M3),
])
def test_one_token_large_layers(n, k, log2c, enc, mode):
    dmode, omode = MODES[mode]
    nst = Nested(workloads.weight_fp16(n, k, seed=n), log2c, slot_seed=3, enc=enc)
    x = workloads.activations_fp16(1, k, seed=4)
    ref = oracle.linear(omode, u16(x), nst.hi_ref, nst.res_ref if mode == "full" else None,
                        enc=enc)
    assert_close(dps.linear(x.to(DEV), nst.nw, dmode), ref)


@pytest.mark.parametrize("numel", [8 * 255 + 3, 8 * 1024, 8 * 1027 + 5])
def test_encoding_choice_sees_every_vector(numel):
    w = workloads.weight_fp16(1, numel, seed=9).reshape(-1).contiguous().to(DEV)
    last = (numel - 1) // 8
    got = []
    for vec in range(last + 1):
        at = min(8 * vec + vec % 8, numel - 1)
        keep = w[at].clone()
        w[at] = -1.875
        got.append(dps.select_enc(w))
        w[at] = keep
    assert bool((torch.cat([g.reshape(1) for g in got]) == dps.ENC_E5M2).all())
    assert dps.select_enc(w).item() == dps.ENC_E4M3
