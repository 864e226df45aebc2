"""GPU parity of the fp32 kernels of few rows that form their own normalised operand, and of attention over heads of at
most 32 elements: head widths around the lanes' split, contexts around a chunk of 64 keys, one to five rows, hidden states
at an address that is only 4-byte aligned."""
import numpy as np
import pytest

from oracle import pt_oracle as O
from paper_2602_07306_amd import inputs as I
from tests.helpers import FP32_TOL, assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [8, 16, 24, 32, 40])
@pytest.mark.parametrize("B,S", [(1, 63), (1, 64), (5, 65), (3, 130)])
def test_fp32_rows_with_their_own_norm(hd, B, S):
    from paper_2602_07306_amd import binding as PB
    cfg = I.PTConfig(n_tracks=2, n_layers=2, block_depth=1, d_model=72, n_heads=4, n_kv_heads=2, head_dim=hd, d_ffn=96,
                     vocab=136, max_batch=B, max_seq=S + 3, dtype=I.PT_F32)
    W = I.make_weights(cfg, 47)
    tokens = I.make_tokens(47, B, S, cfg.vocab)
    st = O.PTState(cfg, B, cfg.max_seq)
    ref = O.pt_prefill(cfg, W, st, tokens=tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(47)
    model._kv.fill_(255)   # NaN everywhere
    lg, _ = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_LAST)
    torch.cuda.synchronize()
    assert_close(lg.cpu().numpy(), ref["logits"][:, -1], FP32_TOL, "prefill logits")
    rng = np.random.default_rng(47)
    for step in range(3):
        x = rng.standard_normal((B, cfg.d_model)).astype(np.float32)
        step_ref = O.pt_decode_step(cfg, W, st, hidden_in=x)
        room = torch.zeros(x.size + 4, dtype=torch.float32, device="cuda")
        off = step + 1                                   # 4, 8, 12 bytes past an aligned address
        room[off:off + x.size] = torch.from_numpy(x).cuda().flatten()
        got, _, _ = model.pt_decode_step(hidden_in=room[off:off + x.size].view(B, cfg.d_model))
        torch.cuda.synchronize()
        assert_close(got.cpu().numpy(), step_ref["logits"], FP32_TOL, "decode step")
    model.close()
