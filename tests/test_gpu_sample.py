"""Most-recent neighbour sampling against a search on the CPU, list by list, bit for bit.

Lists at the edges of the 32-way search (empty, 31 to 33 entries, 32^2 and its neighbours, three levels), more
slots than lanes, query times before, on, between and after the entries, equal times, and a device count
below the maximum (rows past it stay as they were).
"""

import numpy as np
import pytest
import torch

from paper_2608_16305_amd import mtgnn as M
from tests._gpu import log, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

LENGTHS = (0, 1, 2, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025, 1056, 1057, 5000, 33000)


@pytest.mark.parametrize("k", [1, 5, 20, 31, 32, 33, 64])
@pytest.mark.parametrize("ties", [False, True])
def test_sample_recent_list_edges(k, ties):
    log(f"[sample] k {k}, equal times {ties}")
    rng = np.random.default_rng(k + 100 * ties)
    off = np.concatenate([[0], np.cumsum(LENGTHS)]).astype(np.int64)
    n = int(off[-1])
    t = np.concatenate([np.sort(rng.integers(0, max(2, m // 8) if ties else 10 * m + 2, m)) for m in LENGTHS if m])
    t = t.astype(np.float32)
    nbr = rng.integers(0, 1000, n).astype(np.int32)
    eid = rng.permutation(n).astype(np.int32)
    q_node, q_t = [], []
    for i, m in enumerate(LENGTHS):
        at = t[off[i]:off[i + 1]]
        times = [-1.0, 0.0, 1e9] + [float(at[j]) + s for j in {0, m // 3, m // 2, m - 1} if 0 <= j < m for s in (-0.5, 0, 0.5)]
        q_node += [i] * len(times)
        q_t += times
    order = rng.permutation(len(q_node))   # the two queries of a wave are of different lists
    q_node = np.asarray(q_node, np.int32)[order]
    q_t = np.asarray(q_t, np.float32)[order]
    max_q, n_q = len(q_node), len(q_node) - 3
    dev = lambda a: torch.from_numpy(a).cuda()   # noqa: E731
    out = [torch.full((max_q, k), -7, dtype=d, device="cuda") for d in (torch.int32, torch.float32, torch.int32)]
    M.mtgnn_sample_recent(dev(off), dev(nbr), dev(t), dev(eid), len(LENGTHS), dev(q_node), dev(q_t),
                          torch.tensor([n_q], dtype=torch.int32, device="cuda"), max_q, k, *out)
    torch.cuda.synchronize()
    ref = [np.full((max_q, k), -7, a.dtype) for a in (nbr, t, eid)]
    for q in range(n_q):
        lo, hi = off[q_node[q]], off[q_node[q] + 1]
        end = lo + np.searchsorted(t[lo:hi], q_t[q], side="left")
        idx = np.arange(end - 1, max(end - 1 - k, lo - 1), -1)
        for r, a, fill in zip(ref, (nbr, t, eid), (-1, 0, -1)):
            r[q] = fill
            r[q, :idx.size] = a[idx]
    for got, r in zip(out, ref):
        assert np.array_equal(got.cpu().numpy(), r)
