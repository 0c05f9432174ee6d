"""Attention at the edges of its tiles, for every compiled (dtype, d, b):
lengths around the 32-row waves, the 32- and 64-key steps and the block size,
lists of random length in random order, and the dense kernel, against the
oracle.

Tolerances.  bf16: the bars of test_gpu_parity.py.  fp32: outputs are
convex combinations of V (|V| < 6 here), a probability p = 2^x with |x| < 64
carries the rounding of its score (about 64 * 2^-24 * ln 2 = 2.6e-6 relative,
doubled for the normaliser), so |dO| <= 6 * 2 * 2.6e-6 = 3.2e-5; a score's
rounding over the 8 steps of its dot product, 8 * 64 * 2^-25 * ln 2 = 1.1e-5,
and that of the maximum and of the logarithm bound |dlse| by 2e-5.  The oracle
runs in 64 bits here: its own fp32 rounding reaches 1.7e-5 in lse.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import proxyattn_oracle as O
from paper_2509_24745_amd.synth import Structure, Workload

pytestmark = pytest.mark.gpu

LENGTHS = [1, 31, 33, 64, 65, 97, 129, 191, 257, 390]


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_attention_at_tile_edges(dtype, d, b, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as U
    monkeypatch.setattr(O, "F32", np.float64)
    tol_o, tol_l = (2e-2, 4e-3) if dtype == "bf16" else (3.2e-5, 2e-5)
    worst = [0.0, 0.0]
    for n in LENGTHS:
        wl = Workload(name="t", seq_len=n, num_q_heads=4, num_kv_heads=2, head_dim=d, block_size=b,
                      num_proxy_groups=2, stride=4, dtype=dtype, seed=n,
                      structure=Structure(rank=8, hot_blocks=1))
        q, k, v = U.inputs(wl)
        prob = U.problem_of(wl)
        mq = prob.num_blocks
        rng = np.random.default_rng(n)
        bc = np.zeros((4, mq), np.int32)
        bi = np.full((4, mq, mq), -1, np.int32)
        for i in range(4):
            for m in range(mq):
                kk = int(rng.integers(1, m + 2))
                bi[i, m, :kk] = rng.permutation(m + 1)[:kk]
                bc[i, m] = kk
        for lists in ((bc, bi), O.full_causal_lists(n, 4, b)):
            dense = lists[0] is not bc
            out, lse = (U.run_attention(prob, q, k, v, dense=True) if dense
                        else U.run_attention(prob, q, k, v, *lists))
            ref, ref_lse = O.block_sparse_attention(q, k, v, *lists, b, O.default_scale(d))
            worst = [max(worst[0], float(np.max(np.abs(out - ref)))),
                     max(worst[1], float(np.max(np.abs(lse - ref_lse))))]
            assert worst[0] <= tol_o and worst[1] <= tol_l, (n, dense, worst)
    print(f"\n[{dtype} d={d} b={b}] max|dO|={worst[0]:.2e} max|dlse|={worst[1]:.2e}", flush=True)
