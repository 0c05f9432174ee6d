"""Block scores of long sequences (more than 256 key blocks, where the block
maxima are taken by groups of lanes), every b' = b / s, rows ending inside a
block, against a 64-bit reference.  One head, so the pooled heads are the
strided inputs.  Tolerance: that of test_gpu_parity.py for block scores."""
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import LOGA_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s", [(64, 4), (64, 2), (64, 1), (128, 4), (128, 1)])
@pytest.mark.parametrize("blocks", [256, 257, 330])
def test_block_scores_of_long_rows(b, s, blocks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_24745_amd import proxyattn as pa
    n = blocks * b - 37
    prob = pa.Problem(seq_len=n, num_q_heads=1, num_kv_heads=1, head_dim=64, block_size=b,
                      num_proxy_groups=1, stride=s, dtype="bf16")
    gen = torch.Generator(device="cuda").manual_seed(blocks * b + s)
    q, k = (torch.randn((n, 1, 64), generator=gen, device="cuda").mul(1.5).to(torch.bfloat16)
            for _ in range(2))
    bufs = pa.Buffers(prob)
    pa.proxyattn_estimate(prob, q, k, bufs.logscore, bufs.mass, bufs.workspace)
    got = bufs.logscore[0].double()
    bp = b // s
    qs, ks = (x[::s, 0].double() for x in (q, k))
    npr = qs.shape[0]
    ref = torch.full((blocks, blocks), float("-inf"), dtype=torch.float64, device="cuda")
    u = torch.arange(npr, device="cuda")
    for m in range(blocks):
        t = torch.arange(m * bp, min((m + 1) * bp, npr), device="cuda")
        x = (qs[t] @ ks.t()) / 8.0
        x.masked_fill_(u[None, :] > t[:, None], float("-inf"))
        x = (x - torch.logsumexp(x, dim=1, keepdim=True)).amax(dim=0)
        x = torch.nn.functional.pad(x, (0, blocks * bp - npr), value=float("-inf"))
        ref[m] = x.reshape(blocks, bp).amax(dim=1)
    assert torch.equal(torch.isneginf(got), torch.isneginf(ref))
    fin = torch.isfinite(ref)
    err = float((got - ref)[fin].abs().max())
    print(f"\n[b={b} s={s} blocks={blocks}] max|dlogA|={err:.2e}", flush=True)
    assert err <= LOGA_TOL, err
