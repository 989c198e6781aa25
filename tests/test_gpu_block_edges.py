"""The prefill with 128-key tiles at the edges of its tiles: sequences that end
inside, at and past a 64-key half (whose K8/V8 buffers then hold no second half
of the last tile), inside and at a query block, against the CPU oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("br", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("N", [1, 17, 63, 64, 65, 127, 128, 129, 192, 193, 320, 449])
def test_prefill_128_key_tiles(orc, dev, br, causal, N):
    import paper_2412_08585_amd as ta
    print(f"prefill blocks br={br} bc=128 causal={causal} N={N}", flush=True)
    B, Hq, Hkv = 2, 4, 2
    g = torch.Generator().manual_seed(1000 * br + N)
    q = torch.randn(B, Hq, N, 128, generator=g).half()
    k = torch.randn(B, Hkv, N, 128, generator=g).half()
    v = torch.randn(B, Hkv, N, 128, generator=g).half()
    k[..., 3] *= 10
    kv = ta.turbo_quantize_kv(k.to(dev), v.to(dev), block_cols=128)
    o, lse = ta.turbo_attn_prefill(q.to(dev), *kv, causal=causal, return_lse=True, block_rows=br,
                                   block_cols=128)
    torch.cuda.synchronize()
    ro, rl = orc.attn_prefill(q, k, v, 1 / np.sqrt(128), causal, block_rows=br, block_cols=128)
    err = np.abs(o.float().cpu().numpy() - ro) / np.abs(ro).max(axis=-1, keepdims=True)
    assert err.max() < 1e-3
    assert np.abs(lse.cpu().numpy() - rl).max() < 1e-4
