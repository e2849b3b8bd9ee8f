"""Attention with keys shared over four waves keeps its bits: the parts are rounded when they are scaled and again when they are added,
whichever thread does either.  Recorded results of both tile-buffer forms, with waves that see no tile and ragged streams among them."""
import hashlib
import os

import numpy as np
import pytest

from paper_2412_11272_amd import binding as wf

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "attention_shared_keys.txt")
CASES = [line.split() for line in open(GOLDEN) if not line.startswith("#")]


@pytest.mark.parametrize("lens,heads,form,digest", CASES, ids=[f"{c[0]}x{c[1]}" for c in CASES])
def test_recorded_bits(lens, heads, form, digest):
    import torch
    lens, heads = [int(v) for v in lens.split(",")], int(heads)
    assert wf.attention_form(heads, lens) == int(form)
    M, d = sum(lens), 64 * heads
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    qkv = np.random.default_rng(1000 + M).standard_normal((M, 3 * d)).astype(np.float32)
    qkv[:, :2 * d] *= 2.0
    out = torch.empty((M, d), dtype=torch.bfloat16, device="cuda")
    wf.op_attention(wf.WF_PRECISION_BF16, torch.from_numpy(qkv).bfloat16().cuda(), out, cu, heads)
    assert hashlib.sha256(out.view(torch.int16).cpu().numpy().tobytes()).hexdigest() == digest
