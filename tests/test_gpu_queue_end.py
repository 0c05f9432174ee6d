"""The attention work queues where a launch has about as many items as
resident workgroups (1024 of them at bf16, d 64, b 64 on 256 CUs): the first
items by workgroup number, the rest from the queues, and the way out."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _layer(n, hq, hkv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_24745_amd import proxyattn as pa
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((n, h, 64), generator=gen, device="cuda").to(torch.bfloat16)
               for h in (hq, hkv, hkv))
    prob = pa.Problem(seq_len=n, num_q_heads=hq, num_kv_heads=hkv, head_dim=64, block_size=64,
                      num_proxy_groups=1)
    return pa, prob, q, k, v


def _dense(pa, prob, q, k, v):
    kvb = torch.empty(pa.proxyattn_kv_blocked_size(prob), dtype=torch.uint8, device="cuda")
    ws = torch.empty(pa.proxyattn_blocked_workspace_size(prob), dtype=torch.uint8, device="cuda")
    out = torch.full((prob.seq_len, prob.num_q_heads, 64), float("nan"), dtype=torch.bfloat16,
                     device="cuda")
    lse = torch.full((prob.num_q_heads, prob.seq_len), float("nan"), device="cuda")
    pa.proxyattn_prepare_kv(prob, k, v, kvb)
    pa.proxyattn_dense_prefill_blocked(prob, q, kvb, out, lse, ws)
    torch.cuda.synchronize()
    return out, lse, ws


@pytest.mark.parametrize("rows", [1, 7, 24])
def test_few_items_touch_no_counter(rows):
    """With no more items than workgroups nothing is taken from a queue: the
    counters, cleared by the call, stay zero."""
    out, lse, ws = _dense(*_layer(64 * rows - 3, 32, 8))
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
    assert int(ws.view(torch.int32).abs().max()) == 0


@pytest.mark.parametrize("rows", [31, 32, 33, 64])
def test_around_the_resident_workgroups(rows):
    """Every item is computed once: bitwise the same heads in launches of half
    the heads (whole lists on both sides)."""
    pa, prob, q, k, v = _layer(64 * rows - 3, 32, 8)
    out, lse, _ = _dense(pa, prob, q, k, v)
    for h in (0, 1):
        half = pa.Problem(seq_len=prob.seq_len, num_q_heads=16, num_kv_heads=4, head_dim=64,
                          block_size=64, num_proxy_groups=1)
        qs, ks, vs = (x[:, h * x.shape[1] // 2:(h + 1) * x.shape[1] // 2].contiguous()
                      for x in (q, k, v))
        o, l, _ = _dense(pa, half, qs, ks, vs)
        assert torch.equal(o, out[:, 16 * h:16 * h + 16])
        assert torch.equal(l, lse[16 * h:16 * h + 16])
