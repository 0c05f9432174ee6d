"""fp32 operands as three bf16 terms: what a product leaves out, and the range
in which the terms add up to the operand.

Bounds.  Units of 2^-24 of the product.  With one operand's first term rounded
and the other's truncated the three products left out come to less than 2
units; with both truncated to nearly 4 (operands like 0x3f80ff80, whose second
terms are then 2^-7 and third terms 2^-16, all of one sign).  Of the roundings,
the last addition to the accumulator may truncate (2 units), the five before it
act on sums below 2^-6 (0.2 units), and the normaliser's multiplication by ln 2
rounds (1 unit); the scale is chosen so that the other factor is exactly 1."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

F = np.float32
SCALE = F(math.log(2.0))          # times log2(e) in fp32: exactly 1
ROUNDINGS = 2.0 + 0.2 + 1.0


def _near(x):                      # to bf16, nearest even
    u = x.view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + (u >> 16 & 1)) & 0xffff0000).astype(np.uint32).view(F)


def _terms(x, near):
    hi = _near(x) if near else (x.view(np.uint32) & np.uint32(0xffff0000)).view(F)
    mid = _near(x - hi)
    return [t.astype(np.float64) for t in (hi, mid, _near(x - hi - mid))]


def _left_out(x, y, near):
    """What the six products leave out, in units of the whole product."""
    a, b = _terms(x, near), _terms(y, False)
    kept = sum(a[i] * b[j] for i in range(3) for j in range(3) if i + j <= 2)
    exact = x.astype(np.float64) * y.astype(np.float64)
    return np.abs(kept - exact) / np.abs(exact) * 2.0 ** 24


def _aligned():
    """Operands near a power of two whose truncated terms are as large as they
    get: leading bits 0x3f80 .. 0x3f83, then 0xff80 and its neighbours."""
    lead = np.arange(0x3f80, 0x3f84, dtype=np.uint32) << np.uint32(16)
    tail = np.arange(0xff78, 0xff89, dtype=np.uint32)
    return (lead[:, None] | tail[None]).reshape(-1).view(F)


def test_left_out_products_and_exact_range():
    rng = np.random.default_rng(0)
    x, y = (rng.integers(0x3f800000, 0x40000000, 1 << 20, dtype=np.uint32).view(F) for _ in range(2))
    assert _left_out(x, y, True).max() < 2.0
    p = _aligned()
    a, b = (z.reshape(-1) for z in np.meshgrid(p, p))
    assert _left_out(a, b, True).max() < 2.0
    assert 3.5 < _left_out(a, b, False).max() < 4.0
    for near in (True, False):
        bits = rng.integers(0, 0x7f7f0000, 1 << 20, dtype=np.uint32)
        bits |= rng.integers(0, 2, bits.size, dtype=np.uint32) << np.uint32(31)
        v = np.concatenate([bits, bits % np.uint32(20 << 23)]).astype(np.uint32).view(F)
        off = np.abs(sum(_terms(v, near)) - v.astype(np.float64))
        assert off[np.abs(v) >= 2.0 ** -110].max() == 0.0
        assert 0.0 < off.max() <= 2.0 ** -134


def _one_token(q, k, v):
    """Attention of a single token per head: lse = scale * q . k, out = v."""
    from paper_2509_24745_amd import proxyattn as pa
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    heads, d = q.shape
    prob = pa.Problem(seq_len=1, num_q_heads=heads, num_kv_heads=heads, head_dim=d, block_size=64,
                      num_proxy_groups=1, dtype="fp32", softmax_scale=float(SCALE))
    b = pa.Buffers(prob)
    pa.proxyattn_dense_prefill(prob, *(torch.from_numpy(x[None]).cuda() for x in (q, k, v)), b.out,
                               b.lse, b.workspace)
    torch.cuda.synchronize()
    return b.out[0].cpu().numpy(), b.lse[:, 0].double().cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
def test_single_products(d):
    """One non-zero product per head.  The aligned operands' rounded terms
    leave out next to nothing, so only the roundings are left: with both
    operands truncated they exceed the bound."""
    rng = np.random.default_rng(d)
    p = _aligned()
    a, b = (z.reshape(-1)[:4096] for z in np.meshgrid(p, p))
    assert _left_out(a, b, True).max() < 0.1 and _left_out(a, b, False).max() > 3.5
    x, y = (rng.uniform(1, 2, 4096).astype(F) for _ in range(2))
    # queries past the largest bf16, whose first term stays at it
    top = rng.integers(0x7f7f8000, 0x7f800000, 4096, dtype=np.uint32).view(F)
    for u, w, left in ((a, b, 0.1), (x, y, 2.0), (top, y * F(2.0 ** -109), 4.0)):
        q, k = (np.zeros((u.size, d), F) for _ in range(2))
        q[:, 5], k[:, 5] = u, w
        _, lse = _one_token(q, k, np.ones_like(q))
        ref = u.astype(np.float64) * w.astype(np.float64) * float(F(math.log(2.0)))
        err = float(np.max(np.abs(lse / ref - 1.0)) * 2.0 ** 24)
        print(f"\n[d={d}] largest error {err:.2f} units, bound {left + ROUNDINGS:.1f}", flush=True)
        assert err <= left + ROUNDINGS


@pytest.mark.gpu
def test_values_pass_through():
    """With one visible key the probability is 1 and the output the value,
    bit for bit from 2^-110 up and within 2^-134 below."""
    rng = np.random.default_rng(7)
    q = np.zeros((4096, 64), F)
    for lo, hi in ((17 << 23, 0x7f800000), (0, 17 << 23)):
        bits = rng.integers(lo, hi, q.shape, dtype=np.uint32)
        v = (bits | rng.integers(0, 2, q.shape, dtype=np.uint32) << np.uint32(31)).view(F)
        out, _ = _one_token(q, q, v)
        off = np.abs(out.astype(np.float64) - v.astype(np.float64)).max()
        assert off <= (0.0 if lo else 2.0 ** -134)
