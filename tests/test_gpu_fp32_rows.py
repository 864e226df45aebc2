"""GPU parity of the fp32 model where its GEMMs change kernels: one row, the remainder of a group of rows, the sizes on
both sides of the rule, head widths of 32 and more and a context past one chunk of 64 keys, over a cache of NaN bytes."""
import dataclasses

import numpy as np
import pytest

from oracle import pt_oracle as O
from paper_2602_07306_amd import inputs as I
from tests.helpers import FP32_TOL, assert_close, oracle_prefill

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,heads,kv_heads", [(32, 4, 4), (24, 4, 2), (80, 2, 1), (8, 2, 2)])
@pytest.mark.parametrize("B,S", [(1, 1), (1, 6), (2, 33), (3, 67), (1, 130)])
def test_fp32_rows(hd, heads, kv_heads, B, S):
    from paper_2602_07306_amd import binding as PB
    cfg = dataclasses.replace(I.config_tiny(), n_heads=heads, n_kv_heads=kv_heads, head_dim=hd, max_batch=3, max_seq=133)
    W = I.make_weights(cfg, 51)
    tokens = I.make_tokens(51, B, S, cfg.vocab)
    ref, st = oracle_prefill(cfg, W, tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(51)
    model._kv.fill_(255)   # NaN everywhere
    lg, _ = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL)
    torch.cuda.synchronize()
    assert_close(lg.cpu().numpy().reshape(B, S, -1), ref["logits"], FP32_TOL, "logits")
    nxt = tokens[:, 0].copy()
    for _ in range(3):
        want = O.pt_decode_step(cfg, W, st, tokens=nxt)["logits"]
        step, _, _ = model.pt_decode_step(torch.from_numpy(nxt).cuda())
        torch.cuda.synchronize()
        assert_close(step.cpu().numpy(), want, FP32_TOL, "decode step")
    model.close()
