"""Attention with the lists of a launch of few items (at most 256, of at least
8 block rows) split over two wave groups, on both sides of that line: 7 and 8
block rows, and the same heads repeated until there are too many items.
Against the oracle, at the edges of the tiles, for every (dtype, d, b), with
lists down to one block (an empty second group).
Tolerances: those of test_gpu_tiles.py (the join adds two roundings of 2^-24
to each sum, far below them)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import proxyattn_oracle as O
from paper_2509_24745_amd.synth import Structure, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_split_and_whole_lists(dtype, d, b, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as U
    monkeypatch.setattr(O, "F32", np.float64)
    tol_o, tol_l = (2e-2, 4e-3) if dtype == "bf16" else (3.2e-5, 2e-5)
    for n in (7 * b, 7 * b + 1, 8 * b + 33, 11 * b - 31):
        wl = Workload(name="t", seq_len=n, num_q_heads=4, num_kv_heads=2, head_dim=d, block_size=b,
                      num_proxy_groups=2, stride=4, dtype=dtype, seed=n,
                      structure=Structure(rank=8, hot_blocks=1))
        q, k, v = U.inputs(wl)
        mq = U.problem_of(wl).num_blocks
        rng = np.random.default_rng(n)
        bc = np.zeros((4, mq), np.int32)
        bi = np.full((4, mq, mq), -1, np.int32)
        for i in range(4):
            for m in range(mq):
                kk = 1 if (i + m) % 3 == 0 else int(rng.integers(1, m + 2))
                bi[i, m, :kk] = rng.permutation(m + 1)[:kk]
                bc[i, m] = kk
        for lists in ((bc, bi), O.full_causal_lists(n, 4, b)):
            dense = lists[0] is not bc
            ref, ref_lse = O.block_sparse_attention(q, k, v, *lists, b, O.default_scale(d))
            # the most repeats with 256 items, and one more
            for r in (1, 256 // (4 * mq), 256 // (4 * mq) + 1):
                prob = U.problem_of(wl.replace(num_q_heads=4 * r, num_kv_heads=2 * r))
                x = [np.tile(t, (1, r, 1)) for t in (q, k, v)]
                out, lse = (U.run_attention(prob, *x, dense=True) if dense else
                            U.run_attention(prob, *x, *(np.tile(t, (r,) + (1,) * (t.ndim - 1))
                                                        for t in lists)))
                # (a head's list is that of its place among the four: tiling
                # keeps Hq / Hkv = 2)
                do = float(np.max(np.abs(out - np.tile(ref, (1, r, 1)))))
                dl = float(np.max(np.abs(lse - np.tile(ref_lse, (r, 1)))))
                assert do <= tol_o and dl <= tol_l, (n, dense, r, do, dl)
