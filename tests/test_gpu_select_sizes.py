"""Budgets and lists where the sorts change form: block counts around every
power of two up to the largest a wave sorts in registers and past it, scores
with ties, infinities and zeros of both signs, against plain NumPy.  Lists are
compared exactly; counts with the library's sums replayed in fp32 (64-block
butterflies, groups in order, shares sorted, Hillis-Steele prefixes)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

F = np.float32
HQ, G = 6, 2


def _count(mass, gamma):
    nk = mass.size
    pad = -(-nk // 64) * 64
    t = np.zeros(pad, F)
    t[:nk] = mass
    t = t.reshape(-1, 64)
    for o in (32, 16, 8, 4, 2, 1):
        t = t + t[:, np.arange(64) ^ o]
    total = F(0)
    for x in t[:, 0]:
        total = F(total + x)
    s = np.zeros(pad, F)
    s[:nk] = np.sort(mass / total)[::-1]
    s = s.reshape(-1, 64)
    incl = s.copy()
    o = 1
    while o < 64:
        incl[:, o:] = incl[:, o:] + incl[:, :-o].copy()
        o *= 2
    base = F(0)
    for r in range(s.shape[0]):
        excl = np.concatenate([[F(0)], incl[r, :-1]])
        run = (base + excl).astype(F) + s[r]
        hit = np.nonzero((run >= F(gamma)) & (64 * r + np.arange(64) < nk))[0]
        if hit.size:
            return 64 * r + int(hit[0]) + 1
        base = F(base + incl[r, 63])
    return nk


@pytest.mark.parametrize("nk", [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 513, 1001, 1024,
                                1025, 2047, 2048, 2049])
def test_budgets_and_lists(nk):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_24745_amd import proxyattn as pa
    prob = pa.Problem(seq_len=64 * nk - 7, num_q_heads=HQ, num_kv_heads=2, head_dim=64,
                      block_size=64, num_proxy_groups=G, stride=4)
    rng = np.random.default_rng(nk)
    sc = rng.standard_normal((G, nk, nk)).astype(F)
    sc[rng.random(sc.shape) < 0.3] = F(-1.5)                 # ties
    sc[rng.random(sc.shape) < 0.02] = F(-0.0)
    sc[rng.random(sc.shape) < 0.02] = F(0.0)
    sc[rng.random(sc.shape) < 0.01] = F(np.inf)
    sc[rng.random(sc.shape) < 0.01] = -F(np.inf)
    sc = np.where(np.tril(np.ones((nk, nk), bool)), sc, -F(np.inf)).astype(F)
    mass = (rng.random((HQ, nk)) ** 6).astype(F)
    mass[0] = 1.0                                            # all shares equal
    mass[1, rng.random(nk) < 0.5] = 0.0
    mass[1, nk // 2] = 1.0
    dev = "cuda"
    s, m = torch.from_numpy(sc).to(dev), torch.from_numpy(mass).to(dev)
    hc = torch.zeros(HQ, dtype=torch.int32, device=dev)
    bc = torch.zeros((HQ, nk), dtype=torch.int32, device=dev)
    bi = torch.zeros((HQ, nk, nk), dtype=torch.int32, device=dev)
    # order of the float's bits: -0.0 before +0.0 (ascending), as the library's keys
    u = sc.view(np.uint32).astype(np.int64)
    key = np.where(u >> 31 == 1, 0xFFFFFFFF - u, u + 0x80000000)
    rank = np.argsort(-key, axis=2, kind="stable")           # ties to the lower index
    rows = np.arange(1, nk + 1)
    for gamma in (0.5, 0.97):
        pa.proxyattn_select_budget(prob, s, m, gamma, 0, hc, bc, bi)
        counts, cnt, idx = hc.cpu().numpy(), bc.cpu().numpy(), bi.cpu().numpy()
        if nk <= 1024:
            assert counts.tolist() == [_count(mass[i], gamma) for i in range(HQ)]
        for i in range(HQ):
            want = np.minimum(counts[i], rows)
            assert np.array_equal(cnt[i], want)
            # candidates past the diagonal are -inf with a higher index, so
            # they rank behind every causal one
            r = rank[i // (HQ // G)]
            ref = np.where(np.arange(nk)[None] < want[:, None], r, -1)
            causal = ref <= rows[:, None] - 1
            assert causal.all() and np.array_equal(idx[i], ref)
