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


@pytest.mark.parametrize("rows", [200, 256])
@pytest.mark.parametrize("dtype,d,b", [("bf16", 64, 64), ("fp32", 64, 64), ("bf16", 128, 64),
                                       ("fp32", 64, 128)])
def test_long_lists_and_empty_rows(dtype, d, b, rows):
    """One head of up to 256 block rows: halves of more than 64 entries (a wave
    holds its list 64 entries at a time), and rows with an empty list between
    long ones (out = 0, lse = -inf).  The reference runs in 64 bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_24745_amd import proxyattn as pa
    tol_o, tol_l = (2e-2, 4e-3) if dtype == "bf16" else (3.2e-5, 2e-5)
    n = rows * b - 29
    prob = pa.Problem(seq_len=n, num_q_heads=1, num_kv_heads=1, head_dim=d, block_size=b,
                      num_proxy_groups=1, dtype=dtype)
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    q, k, v = (torch.randn((n, 1, d), generator=gen, device="cuda").to(prob.torch_dtype)
               for _ in range(3))
    rng = np.random.default_rng(rows)
    bc = np.zeros((1, rows), np.int32)
    bi = np.full((1, rows, rows), -1, np.int32)
    for m in range(rows):
        kk = 0 if m % 7 == 3 else int(rng.integers(min(m + 1, 130), m + 2))
        bi[0, m, :kk] = rng.permutation(m + 1)[:kk]
        bc[0, m] = kk
    bc, bi = torch.from_numpy(bc).cuda(), torch.from_numpy(bi).cuda()
    bufs = pa.Buffers(prob)

    def reference(lists):   # out [n, d], lse [n]
        qd, kd, vd = (x[:, 0].double() for x in (q, k, v))
        u = torch.arange(n, device="cuda")
        out, lse = torch.zeros(n, d, dtype=torch.float64, device="cuda"), torch.zeros(n, device="cuda").double()
        for m in range(rows):
            t = u[m * b:(m + 1) * b]
            keep = torch.zeros(rows, dtype=torch.bool, device="cuda")
            if lists:
                keep[bi[0, m, :int(bc[0, m])].long()] = True
            else:
                keep[:m + 1] = True
            mask = keep[u // b][None, :] & (u[None, :] <= t[:, None])
            s = ((qd[t] @ kd.t()) * prob.scale).masked_fill(~mask, float("-inf"))
            lse[t] = torch.logsumexp(s, dim=1)
            out[t] = torch.nan_to_num(torch.softmax(s, dim=1)) @ vd
        return out, lse

    for lists in (True, False):
        bufs.out.fill_(float("nan"))
        bufs.lse.fill_(float("nan"))
        if lists:
            pa.proxyattn_block_sparse_prefill(prob, q, k, v, bc, bi, bufs.out, bufs.lse, bufs.workspace)
        else:
            pa.proxyattn_dense_prefill(prob, q, k, v, bufs.out, bufs.lse, bufs.workspace)
        out, lse = bufs.out[:, 0].double(), bufs.lse[0].double()
        ref, ref_lse = reference(lists)
        empty = torch.isneginf(ref_lse)
        assert int(empty.sum()) == (int((bc == 0).sum()) * b - (29 if int(bc[0, -1]) == 0 else 0)
                                    if lists else 0)
        assert torch.equal(torch.isneginf(lse), empty) and not out[empty].any()
        do = float((out - ref).abs().max())
        dl = float((lse - ref_lse)[~empty].abs().max())
        print(f"\n[{dtype} d={d} b={b} rows={rows} lists={lists}] |dO|={do:.2e} |dlse|={dl:.2e}",
              flush=True)
        assert do <= tol_o and dl <= tol_l, (lists, do, dl)
