"""The routing tables at the edges of the ranking kernel (waves of 64, sixteen of them, eight rounds in flight) and of the prefix sums (1 to 256 experts,
one local expert to all of them), against a stable sort."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,n_local", [(0, 8, 2), (1, 2, 1), (31, 2, 2), (32, 64, 64), (33, 65, 5), (511, 255, 1), (512, 256, 64), (513, 256, 4), (4096, 16, 2), (4127, 12, 3)])
@pytest.mark.parametrize("skew", [False, True])
def test_plan_is_a_stable_sort(T, E, n_local, skew):
    from paper_2411_15871_amd import dhelix as dh
    rng = np.random.default_rng(T * 300 + E)
    first = rng.integers(0, E if not skew else min(E, 2), T)
    idx = np.stack([first, (first + rng.integers(1, E, T)) % E], axis=1).astype(np.int32).reshape(-1)
    n = max(1, 2 * T)
    sizes = dict(rank=n, dest=n, src_tok=n, send_of_recv=n, recv_of_send=n, counts=E, offsets=E + 1, recv_start=E, group_rows=n_local)
    ts = {k: torch.full((v,), -7, dtype=torch.int32, device="cuda") for k, v in sizes.items()}
    tb = dh.moe_tables(**ts)
    dh.dh_moe_plan(T, E, n_local, torch.from_numpy(idx).cuda() if T else None, tb)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy()[:2 * T] if v.numel() == n and k not in ("counts", "offsets", "recv_start", "group_rows") else v.cpu().numpy() for k, v in ts.items()}
    counts = np.bincount(idx, minlength=E)
    order = np.argsort(idx, kind="stable")
    dest = np.empty(2 * T, np.int64); dest[order] = np.arange(2 * T)
    offsets = np.concatenate([[0], np.cumsum(counts)])
    perm = [s * n_local + l for l in range(n_local) for s in range(E // n_local)]
    recv_start = np.empty(E, np.int64); recv_start[perm] = np.concatenate([[0], np.cumsum(counts[perm])[:-1]])
    rank = dest - offsets[idx]
    assert np.array_equal(got["counts"], counts) and np.array_equal(got["offsets"], offsets) and np.array_equal(got["recv_start"], recv_start)
    assert np.array_equal(got["group_rows"], counts.reshape(E // n_local, n_local).sum(axis=0))
    assert np.array_equal(got["rank"], rank) and np.array_equal(got["dest"], dest) and np.array_equal(got["src_tok"], order >> 1)
    recv = recv_start[idx] + rank
    ros = np.empty(2 * T, np.int64); ros[dest] = recv
    sor = np.empty(2 * T, np.int64); sor[recv] = dest
    assert np.array_equal(got["recv_of_send"], ros) and np.array_equal(got["send_of_recv"], sor)
