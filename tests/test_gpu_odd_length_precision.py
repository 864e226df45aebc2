"""GPU: what a prompt keeps in 32 bits when its length is no multiple of 32, compared with the shape-generic kernels, which
hold probabilities in fp32 and read the rotary table at every position.  The model is one layer whose output projection
is the identity and whose feed-forward network adds nothing, so the hidden states minus the input are the attention
output."""
import numpy as np
import pytest

from paper_2602_07306_amd import inputs as I
from tests.helpers import small_bf16_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def one_layer(hd, heads, kv_heads, B, S, wq, wk, wv):
    from paper_2602_07306_amd import binding as PB
    d = heads * hd
    cfg = small_bf16_config(n_tracks=1, n_layers=1, block_depth=1, d_model=d, n_heads=heads, n_kv_heads=kv_heads, head_dim=hd, max_batch=B, max_seq=S)
    model = PB.PTModel(cfg)
    model.pt_init_weights(3)
    for name, w in (("wq", wq), ("wk", wk), ("wv", wv), ("wo", np.eye(d, dtype=np.float32)),
                    ("wd", np.zeros((cfg.d_ffn, d), np.float32))):
        model.pt_set_weight(name, 0, 0, w)
    return PB, model


@pytest.mark.parametrize("hd,heads,kv_heads", [(64, 4, 2), (128, 2, 1)])
@pytest.mark.parametrize("B,S", [(4, 31), (2, 33), (3, 100), (1, 197), (1, 1000)])
def test_probabilities_stay_in_32_bits(hd, heads, kv_heads, B, S):
    rng = np.random.default_rng(S)
    d = heads * hd
    # every column of the projections picks one element of the normed input: queries, keys and values are the same numbers
    # on both paths, and scores are about N(0, 1), so that many keys carry weight
    wq, wk, wv = (np.eye(d, dtype=np.float32)[:, rng.permutation(d)[:n * hd]] for n in (heads, kv_heads, kv_heads))
    PB, model = one_layer(hd, heads, kv_heads, B, S, wq, wk, wv)
    x = torch.from_numpy(rng.standard_normal((B, S, d)).astype(np.float32)).cuda()
    out = []
    for path in (PB.PT_PATH_AUTO, PB.PT_PATH_GENERIC):
        model.pt_set_kernel_path(path)
        hid = model.pt_prefill(hidden_in=x, logits_mode=PB.PT_LOGITS_NONE, want_hidden=True)[1]
        torch.cuda.synchronize()
        out.append((hid.double() - x.double()).cpu().numpy().reshape(B, S, d)[:, 1:])   # position 0 sees one key: no rounding
    model.close()
    # Both sum the terms in fp32, in another order: 1e-6 of the result, which moves one rounding to bf16 in about a
    # thousand by a unit: 2^-8 times the root of that share is 1.2e-4.  Probabilities rounded to bf16 shift every term
    # by up to 2^-9 of itself and with it nearly every rounding: about 2e-3.
    err = np.linalg.norm(out[0] - out[1]) / np.linalg.norm(out[1])
    assert err < 3e-4, err


@pytest.mark.parametrize("hd,heads,kv_heads", [(64, 4, 4), (128, 2, 2)])
@pytest.mark.parametrize("B,S", [(5, 31), (3, 100), (1, 1000)])
def test_keys_are_rotated_by_the_table(hd, heads, kv_heads, B, S):
    d = heads * hd
    # every projected element is one product, and the upper half of a head is zero: a rotated key is a single product
    # with the table's cosine or sine, so that every kernel that reads the table leaves the same bytes in the cache
    half = np.tile(np.concatenate([np.ones(hd // 2), np.zeros(hd // 2)]), kv_heads).astype(np.float32)
    PB, model = one_layer(hd, heads, kv_heads, B, S, np.eye(d, dtype=np.float32), np.diag(half), np.eye(d, dtype=np.float32))
    x = torch.from_numpy(np.random.default_rng(S).standard_normal((B, S, d)).astype(np.float32)).cuda()
    cache = []
    for path in (PB.PT_PATH_AUTO, PB.PT_PATH_GENERIC):
        model.pt_set_kernel_path(path)
        model._kv.zero_()
        model.pt_prefill(hidden_in=x, logits_mode=PB.PT_LOGITS_NONE)
        torch.cuda.synchronize()
        cache.append(model._kv.clone())
    model.close()
    assert bool((cache[1] != 0).any())
    differing = int((cache[0] != cache[1]).sum())
    assert differing == 0, differing
