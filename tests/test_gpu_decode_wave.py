"""GPU parity of decode attention with one wavefront per head and key range: both head widths, groups of one to eight query
heads, contexts around a tile of 64 keys and around the split into ranges, sequences of different lengths (ranges
without keys among them), over a cache of NaN bytes."""
import numpy as np
import pytest

from oracle import pt_oracle as O
from paper_2602_07306_amd import inputs as I
from tests.helpers import BF16_TOL, assert_close, small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,heads,kv_heads,T,B,S", [
    (128, 4, 4, 2, 8, 62),     # 64 heads of the cache; the steps cross the first tile's end
    (128, 8, 1, 4, 16, 64),    # groups of eight
    (128, 4, 2, 4, 8, 700),    # three ranges of 256 keys
    (128, 2, 2, 8, 32, 129),   # 512 heads, one range
    (64, 4, 4, 4, 32, 385),    # 512 heads of 64 up to 512 keys: the workgroup form
    (64, 4, 4, 4, 32, 512),    # ... and past them
    (64, 4, 4, 5, 32, 191),    # 640 of them, the fourth tile begins
    (128, 4, 4, 2, 24, 320),   # 192 heads, one range: fewer than six keys a head
    (64, 16, 16, 1, 64, 30),   # 1024 of them, short
])
@pytest.mark.parametrize("ragged", [False, True])
def test_decode_by_wavefronts(hd, heads, kv_heads, T, B, S, ragged):
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_tracks=T, n_layers=1, block_depth=1, d_model=128, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd,
                            d_ffn=128, vocab=256, max_batch=B, max_seq=S + 4)
    W = I.make_weights(cfg, 53)
    tokens = I.make_tokens(53, B, S, cfg.vocab)
    lens = [1 + (7 * b + S - 1) % S for b in range(B)] if ragged else [S] * B
    st = O.PTState(cfg, B, cfg.max_seq)
    if ragged:
        O.pt_prefill(cfg, W, st, tokens=tokens, lengths=np.array(lens))
    else:
        O.pt_prefill(cfg, W, st, tokens=tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(53)
    model._kv.fill_(255)   # bf16 NaN everywhere
    if ragged:
        flat = np.concatenate([tokens[b, :n] for b, n in enumerate(lens)])
        model.pt_prefill_ragged(lens, tokens=torch.from_numpy(flat).cuda(), logits_mode=PB.PT_LOGITS_NONE)
    else:
        model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_NONE)
    nxt = tokens[:, 0].copy()
    for _ in range(3):
        want = O.pt_decode_step(cfg, W, st, tokens=nxt)["logits"]
        got, _, _ = model.pt_decode_step(torch.from_numpy(nxt).cuda())
        torch.cuda.synchronize()
        assert_close(got.cpu().numpy(), want, BF16_TOL, "decode step")
    model.close()
