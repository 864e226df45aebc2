"""GPU parity of the square GEMM tiles (256 x 256 and 128 x 128), each forced for every GEMM that it covers: rows around the
tiles' edges, the shortest K (two and four K steps of 64), K that is no multiple of four steps, a workgroup with several
tiles of a launch, aligned and odd positions, both head widths, grouped KV heads."""
import pytest

from paper_2602_07306_amd import inputs as I
from tests.helpers import BF16_TOL, assert_close, oracle_prefill, path_counts, small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [0, 2])
@pytest.mark.parametrize("B,S,d_model,heads,kv_heads,hd,d_ffn", [
    (1, 65, 128, 2, 2, 64, 128),        # two K steps everywhere; one tile of rows, nearly half empty
    (1, 127, 256, 4, 2, 64, 384),       # four and six K steps, grouped heads
    (2, 128, 128, 2, 2, 64, 640),       # 256 rows: the tiles are full
    (1, 257, 256, 2, 2, 128, 512),      # one row in the second tile, heads of 128, odd positions
    (3, 96, 384, 4, 4, 128, 256),       # 32-row blocks, K of six steps
    (2, 1056, 128, 2, 2, 64, 4096),     # more tiles than workgroups, the last tile of rows a quarter full
    (1, 2111, 256, 2, 1, 128, 2048),    # the same with odd positions and one KV head
    (2, 160, 512, 8, 8, 64, 640),       # four and eight sums of squares per row, added up by the next GEMM
    (1, 330, 1024, 16, 16, 64, 384),    # eight and sixteen, odd positions
])
def test_square_tiles(tile, B, S, d_model, heads, kv_heads, hd, d_ffn):
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_layers=2, block_depth=1, d_model=d_model, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd,
                            d_ffn=d_ffn, vocab=512, max_batch=B, max_seq=S)
    W = I.make_weights(cfg, 43)
    tokens = I.make_tokens(43, B, S, cfg.vocab)
    ref, _ = oracle_prefill(cfg, W, tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(43)
    PB.pt_set_tuning(PB.PT_TUNE_GEMM_TILE_CONFIG, tile)
    try:
        model.pt_profile_reset()
        lg, hid = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL, want_hidden=True)
        torch.cuda.synchronize()
        counts = path_counts(model)
    finally:
        PB.pt_set_tuning(PB.PT_TUNE_GEMM_TILE_CONFIG, -1)
    assert counts["gemm_gateup"][1] == counts["gemm_down"][1] == counts["gemm_out"][1] == cfg.n_layers, counts
    assert_close(lg.cpu().numpy().reshape(B, S, -1), ref["logits"], BF16_TOL, "logits")
    assert_close(hid.cpu().numpy(), ref["hidden"], BF16_TOL, "hidden")
    model.close()


@pytest.mark.parametrize("tile", [0, 2])
@pytest.mark.parametrize("S,vocab", [(66, 136), (193, 392), (257, 264)])   # eight columns in the last tile, rows to match
def test_square_tiles_store_ragged_edges(tile, S, vocab):
    """fp32 results whose last tile is cut in rows and in columns (the head), and nothing behind the last column or row."""
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_layers=1, block_depth=1, d_model=256, n_heads=4, n_kv_heads=4, head_dim=64, d_ffn=256, vocab=vocab, max_batch=1, max_seq=S)
    W = I.make_weights(cfg, 44)
    tokens = I.make_tokens(44, 1, S, cfg.vocab)
    ref, _ = oracle_prefill(cfg, W, tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(44)
    room = torch.full(((S + 2) * vocab,), 7.0, dtype=torch.float32, device="cuda")
    PB.pt_set_tuning(PB.PT_TUNE_GEMM_TILE_CONFIG, tile)
    try:
        lg, _ = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL, logits_out=room[vocab:-vocab].view(S, vocab))
        torch.cuda.synchronize()
    finally:
        PB.pt_set_tuning(PB.PT_TUNE_GEMM_TILE_CONFIG, -1)
    assert_close(lg.cpu().numpy().reshape(1, S, -1), ref["logits"], BF16_TOL, "logits")
    assert bool((room[:vocab] == 7.0).all()) and bool((room[-vocab:] == 7.0).all())
    model.close()


@pytest.mark.parametrize("S,d_model,heads,d_ffn,vocab", [
    (66, 256, 4, 9216, 512),       # gate/up: 576 tiles, K of four steps; workgroups with two and with three of them
    (96, 384, 96, 9216, 512),      # six steps: the four buffers turn on from tile to tile; QKV likewise, in 32-row blocks
    (112, 640, 96, 8448, 512),     # ten steps; QKV of rows of any place, 528 tiles of gate/up
    (70, 256, 4, 256, 73728),      # the head: 576 tiles with results in fp32
])
def test_four_step_tile_with_several_tiles_of_a_launch(S, d_model, heads, d_ffn, vocab):
    """One tile of rows and an odd number of rounds of the 128 x 128 tile: the form with four K steps in flight runs from one
    tile into the next."""
    from paper_2602_07306_amd import binding as PB
    cfg = small_bf16_config(n_tracks=4, n_layers=1, block_depth=1, d_model=d_model, n_heads=heads, n_kv_heads=heads, head_dim=64, d_ffn=d_ffn,
                            vocab=vocab, max_batch=1, max_seq=S)
    W = I.make_weights(cfg, 45)
    tokens = I.make_tokens(45, 1, S, cfg.vocab)
    ref, _ = oracle_prefill(cfg, W, tokens)
    model = PB.PTModel(cfg)
    model.pt_init_weights(45)
    PB.pt_set_tuning(PB.PT_TUNE_GEMM_TILE_CONFIG, 2)
    try:
        lg, hid = model.pt_prefill(torch.from_numpy(tokens).cuda(), logits_mode=PB.PT_LOGITS_ALL, want_hidden=True)
        torch.cuda.synchronize()
    finally:
        PB.pt_set_tuning(PB.PT_TUNE_GEMM_TILE_CONFIG, -1)
    assert_close(lg.cpu().numpy().reshape(1, S, -1), ref["logits"], BF16_TOL, "logits")
    assert_close(hid.cpu().numpy(), ref["hidden"], BF16_TOL, "hidden")
    model.close()
