"""Estimation at the edges of its 64-key steps and their two 32-key tiles:
lengths around the 32-row waves, where a step's second tile is left out (fp32)
or masked, the last tokens' rows not aligned to the blocks, 8 and 9 blocks (the
rows' normalisers change their split there), against a 64-bit reference.  One
head, so the pooled heads are the strided inputs.
Tolerances: those of test_gpu_parity.py for block scores and masses."""
import pytest

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import LOGA_TOL, MASS_RTOL

pytestmark = pytest.mark.gpu

LENGTHS = [1, 16, 31, 32, 33, 63, 64, 65, 96, 97, 129, 161, 255, 300, 512, 513, 1024, 1025]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("b,s", [(64, 4), (64, 1), (128, 2), (128, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_estimate_at_tile_edges(dtype, b, s, d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_24745_amd import proxyattn as pa
    worst = [0.0, 0.0]
    for n in LENGTHS:
        prob = pa.Problem(seq_len=n, num_q_heads=1, num_kv_heads=1, head_dim=d, block_size=b,
                          num_proxy_groups=1, stride=s, dtype=dtype)
        gen = torch.Generator(device="cuda").manual_seed(n)
        q, k = (torch.randn((n, 1, d), generator=gen, device="cuda").mul(1.5).to(prob.torch_dtype)
                for _ in range(2))
        bufs = pa.Buffers(prob)
        pa.proxyattn_estimate(prob, q, k, bufs.logscore, bufs.mass, bufs.workspace)
        mq, bp, rows = prob.num_blocks, b // s, min(b, n)

        def probs(t, u, step):   # log-probabilities of rows t over the keys u <= t
            x = (q[t * step, 0].double() @ k[u * step, 0].double().t()) * prob.scale
            x = x.masked_fill(u[None, :] > t[:, None], float("-inf"))
            return x - torch.logsumexp(x, dim=1, keepdim=True)

        def blocks(x, width, fill):   # [rows, keys] -> [rows, mq, width]
            x = torch.nn.functional.pad(x, (0, mq * width - x.shape[1]), value=fill)
            return x.reshape(x.shape[0], mq, width)

        u = torch.arange(-(-n // s), device="cuda")
        rowmax = blocks(probs(u, u, s), bp, float("-inf")).amax(dim=2)
        logA = torch.stack([rowmax[m * bp:(m + 1) * bp].amax(dim=0) for m in range(mq)])
        u = torch.arange(n, device="cuda")
        mass = blocks(probs(u[n - rows:], u, 1).exp(), b, 0.0).sum(dim=(0, 2))
        got = bufs.logscore[0].double()
        assert torch.equal(torch.isneginf(got), torch.isneginf(logA)), n
        fin = torch.isfinite(logA)
        worst[0] = max(worst[0], float((got - logA)[fin].abs().max()))
        worst[1] = max(worst[1], float((bufs.mass[0].double() - mass).abs().max()) / rows)
        assert worst[0] <= LOGA_TOL and worst[1] <= MASS_RTOL, (n, worst)
    print(f"\n[{dtype} d={d} b={b} s={s}] max|dlogA|={worst[0]:.2e} |dmass|/rows={worst[1]:.2e}",
          flush=True)
