"""GPU parity of prefill at prompt lengths that are no multiple of the attention kernel's 64-key tile, over a KV cache
whose bytes are NaN beforehand: the masked last tile must keep positions that no token has written out of the result."""
import numpy as np
import pytest

from oracle import pt_oracle as O
from paper_2602_07306_amd import inputs as I
from tests.helpers import BF16_TOL, assert_close, oracle_prefill, path_counts, small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,heads,kv_heads", [(64, 4, 2), (128, 2, 2)])
@pytest.mark.parametrize("B,S", [(1, 2), (2, 31), (1, 33), (3, 63), (1, 65), (2, 96), (1, 127), (2, 129), (1, 197), (1, 256)])
def test_prefill_of_any_length_ignores_unwritten_cache(hd, heads, kv_heads, B, S):
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_layers=2, block_depth=1, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd, max_batch=3, max_seq=257)
    W = I.make_weights(cfg, 21)
    tokens = I.make_tokens(21, B, S, cfg.vocab)
    ref, st = oracle_prefill(cfg, W, tokens)
    nxt = np.argmax(ref["logits"][:, -1], -1).astype(np.int32)
    step_ref = O.pt_decode_step(cfg, W, st, tokens=nxt)
    model = PB.PTModel(cfg)
    model.pt_init_weights(21)
    model._kv.fill_(255)   # bf16 NaN everywhere
    model.pt_profile_reset()
    lg, hid = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL, want_hidden=True)
    torch.cuda.synchronize()
    counts = path_counts(model)["attn_prefill"]   # the masked form unless the last tile is full, never the generic kernel
    assert counts[1 if S % 64 == 0 else 2] == cfg.n_layers and sum(counts) == cfg.n_layers, counts
    assert_close(lg.cpu().numpy().reshape(B, S, -1), ref["logits"], BF16_TOL, "prefill logits")
    assert_close(hid.cpu().numpy(), ref["hidden"], BF16_TOL, "prefill hidden")
    step, _, _ = model.pt_decode_step(torch.from_numpy(nxt).cuda())
    torch.cuda.synchronize()
    assert_close(step.cpu().numpy(), step_ref["logits"], BF16_TOL, "decode step")
    model.close()


@pytest.mark.parametrize("hd,heads,kv_heads", [(64, 4, 2), (128, 2, 2)])
@pytest.mark.parametrize("B,S,bad", [(2, 31, 20), (1, 96, 40), (1, 100, 99), (2, 197, 70), (1, 197, 0)])
def test_a_row_of_nan_does_not_reach_earlier_rows(hd, heads, kv_heads, B, S, bad):
    """A hidden state of NaN at one position of sequence 0 makes NaN of that row and the later ones; earlier rows, and the
    other sequence, stay what they are without it."""
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_layers=2, block_depth=1, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd, max_batch=B, max_seq=S)
    model = PB.PTModel(cfg)
    model.pt_init_weights(23)
    x = torch.from_numpy(np.random.default_rng(S).standard_normal((B, S, cfg.d_model)).astype(np.float32)).cuda()
    clean = model.pt_prefill(hidden_in=x, logits_mode=PB.PT_LOGITS_NONE, want_hidden=True)[1].clone()
    y = x.clone()
    y[0, bad] = float("nan")
    hid = model.pt_prefill(hidden_in=y, logits_mode=PB.PT_LOGITS_NONE, want_hidden=True)[1]
    torch.cuda.synchronize()
    assert bool(torch.isnan(hid[0, bad:]).all())
    got = torch.cat([hid[0, :bad], hid[1:].reshape(-1, cfg.d_model)]).cpu().numpy()
    want = torch.cat([clean[0, :bad], clean[1:].reshape(-1, cfg.d_model)]).cpu().numpy()
    if got.size:
        assert np.isfinite(got).all(), np.argwhere(~np.isfinite(got).all(-1)).ravel()
        assert_close(got, want, BF16_TOL, "rows that see no NaN")
    model.close()
