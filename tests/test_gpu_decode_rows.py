"""GPU parity of decode steps of one to four sequences, where the matrix-vector GEMMs run: one, two and four wavefronts
sharing rows along K, odd numbers of 512-wide chunks, RMSNorm from registers and, for wide models, from memory."""
import pytest

from paper_2602_07306_amd import inputs as I
from oracle import pt_oracle as O
from tests.helpers import BF16_TOL, assert_close, path_counts, small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,heads,d_ffn", [(4, 1024, 16, 2048), (8, 512, 8, 1536), (2, 2560, 16, 3072)])
@pytest.mark.parametrize("B", [1, 2, 3, 4])
def test_matrix_vector_decode(T, d, heads, d_ffn, B):
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_tracks=T, n_layers=2, block_depth=1, d_model=d, n_heads=heads, n_kv_heads=heads, d_ffn=d_ffn, max_batch=B, max_seq=16)
    W = I.make_weights(cfg, 43)
    tokens = I.make_tokens(43, B, 9, cfg.vocab)
    st = O.PTState(cfg, B, cfg.max_seq)
    O.pt_prefill(cfg, W, st, tokens=tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(43)
    model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_NONE)
    nxt = tokens[:, 0].copy()
    model.pt_profile_reset()
    for _ in range(2):
        ref = O.pt_decode_step(cfg, W, st, tokens=nxt)
        step, _, _ = model.pt_decode_step(torch.from_numpy(nxt).cuda())
        torch.cuda.synchronize()
        assert_close(step.cpu().numpy(), ref["logits"], BF16_TOL, "decode step")
    counts = path_counts(model)
    assert counts["gemm_out"][3] == 2 * cfg.n_layers and counts["gemm_down"][3] == 2 * cfg.n_layers, counts
    model.close()


@pytest.mark.parametrize("T,d,d_ffn", [(16, 512, 2080), (8, 1536, 4160)])
def test_matrix_vector_workgroups_with_several_units(T, d, d_ffn):
    """More gate/up tiles over all tracks than workgroups: a workgroup walks three units (the last one fewer), of one or
    three 512-wide chunks, and hands its lane sums over between them."""
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_tracks=T, n_layers=1, block_depth=1, d_model=d, n_heads=8, n_kv_heads=2, d_ffn=d_ffn, max_batch=4, max_seq=16)
    assert T * d_ffn // 16 > 2 * 1024
    W = I.make_weights(cfg, 47)
    model = PB.PTModel(cfg)
    model.pt_init_weights(47)
    for B in (1, 2, 3, 4):
        tokens = I.make_tokens(47 + B, B, 5, cfg.vocab)
        st = O.PTState(cfg, B, cfg.max_seq)
        O.pt_prefill(cfg, W, st, tokens=tokens)
        model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_NONE)
        model.pt_profile_reset()
        nxt = tokens[:, 0].copy()
        ref = O.pt_decode_step(cfg, W, st, tokens=nxt)
        step, _, _ = model.pt_decode_step(torch.from_numpy(nxt).cuda())
        torch.cuda.synchronize()
        assert_close(step.cpu().numpy(), ref["logits"], BF16_TOL, "decode step of %d" % B)
        assert path_counts(model)["gemm_gateup"][3] == cfg.n_layers
    model.close()
