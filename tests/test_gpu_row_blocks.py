"""GPU parity of the QKV epilogue where a block of 32 rows is no run of aligned positions: several short sequences in one
block, sequences that end inside it, the last rows of the matrix, one row per sequence, over a cache of NaN bytes."""
import numpy as np
import pytest

from oracle import pt_oracle as O
from paper_2602_07306_amd import inputs as I
from tests.helpers import BF16_TOL, assert_close, small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,heads,kv_heads", [(64, 4, 2), (128, 2, 2)])
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("B,S", [(30, 3), (5, 31), (9, 40), (73, 9), (1, 130)])
def test_row_blocks_of_any_alignment(hd, heads, kv_heads, ragged, B, S):
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_layers=2, block_depth=1, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd, max_batch=B, max_seq=S + 3)
    W = I.make_weights(cfg, 31)
    tokens = I.make_tokens(31, B, S, cfg.vocab)
    lens = [1 + (5 * b + S - 1) % S for b in range(B)] if ragged else [S] * B
    st = O.PTState(cfg, B, cfg.max_seq)
    ref = O.pt_prefill(cfg, W, st, tokens=tokens, lengths=np.array(lens)) if ragged else O.pt_prefill(cfg, W, st, tokens=tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(31)
    model._kv.fill_(255)   # bf16 NaN everywhere
    if ragged:
        flat = np.concatenate([tokens[b, :n] for b, n in enumerate(lens)])
        lg, _ = model.pt_prefill_ragged(lens, tokens=torch.from_numpy(flat).cuda(), logits_mode=PB.PT_LOGITS_ALL)
        want = np.concatenate([ref["logits"][b, :n] for b, n in enumerate(lens)])
    else:
        lg, _ = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL)
        want = ref["logits"].reshape(B * S, -1)
    torch.cuda.synchronize()
    assert_close(lg.cpu().numpy(), want, BF16_TOL, "prefill logits")
    nxt = tokens[:, 0].copy()
    for _ in range(2):
        step_ref = O.pt_decode_step(cfg, W, st, tokens=nxt)
        step, _, _ = model.pt_decode_step(torch.from_numpy(nxt).cuda())
        torch.cuda.synchronize()
        assert_close(step.cpu().numpy(), step_ref["logits"], BF16_TOL, "decode step")
    model.close()
