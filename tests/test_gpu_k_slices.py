"""GPU parity of prefills whose residual GEMMs have too few tiles for the chip: their K is cut into slices that the
normalising kernel adds up.  Rows around the tile's edge, one and several slices, with and without a following norm."""
import numpy as np
import pytest

from paper_2602_07306_amd import inputs as I
from tests.helpers import BF16_TOL, assert_close, oracle_prefill, path_counts, small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# out_rows, down_rows: up to how many rows the rule cuts the out (K = d_model) and the down projection (K = d_ffn): K = 256
# is too short, 512 pays for few rows only, 1024 and more for all of these sizes
@pytest.mark.parametrize("d_model,heads,d_ffn,block_depth,out_rows,down_rows",
                         [(256, 4, 512, 1, 0, 400), (256, 4, 4096, 2, 0, 512), (512, 8, 1024, 1, 200, 512), (256, 4, 256, 2, 0, 0)])
@pytest.mark.parametrize("B,S", [(1, 65), (1, 127), (2, 64), (1, 129), (3, 100), (2, 256)])
def test_prefill_with_k_slices(d_model, heads, d_ffn, block_depth, out_rows, down_rows, B, S):
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_layers=2, block_depth=block_depth, d_model=d_model, n_heads=heads, n_kv_heads=heads, d_ffn=d_ffn, max_batch=3)
    W = I.make_weights(cfg, 41)
    tokens = I.make_tokens(41, B, S, cfg.vocab)
    ref, _ = oracle_prefill(cfg, W, tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(41)
    model.pt_profile_reset()
    lg, hid = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL, want_hidden=True)
    torch.cuda.synchronize()
    counts = path_counts(model)
    assert counts["gemm_out"][1] == cfg.n_layers and counts["gemm_down"][1] == cfg.n_layers, counts
    assert model.pt_profile_paths("rmsnorm")[1] == ((B * S <= out_rows) + (B * S <= down_rows)) * cfg.n_layers
    assert_close(lg.cpu().numpy().reshape(B, S, -1), ref["logits"], BF16_TOL, "logits")
    assert_close(hid.cpu().numpy(), ref["hidden"], BF16_TOL, "hidden")
    model.close()
