"""Sizes at which the kernels around the list scan change their way: edges of samples, buffers and tiles, the smallest
and the largest of each range, against float64 arithmetic of the same operands."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _hr():
    import paper_2507_09138_amd as hr
    return hr


def _index(N, d, nlist, dtype, seed, tables=False, zipf=0.0):
    """An index of random vectors and the arrays it was made from."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cent = torch.randn(nlist, d, generator=g, device="cuda")
    w = torch.arange(1, nlist + 1, dtype=torch.float64) ** -zipf
    sizes = torch.floor((N - nlist) * w / w.sum()).long() + 1
    sizes[0] += N - int(sizes.sum())
    off = torch.zeros(nlist + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(sizes, 0)
    vec = torch.randn(N, d, generator=g, device="cuda").to(dtype)
    ids = torch.randperm(N, generator=g, device="cuda")
    return _hr().IvfIndex(cent, off, vec, ids, row_tables=tables), cent, off, vec, ids, g


def _keys(q, x, metric):
    dots = q @ x.T
    return dots if metric == "ip" else 2 * dots - (x * x).sum(1)


@pytest.mark.parametrize("nlist,nprobe,nq", [(256, 64, 3), (257, 1, 5), (257, 256, 5), (1024, 32, 9), (1025, 512, 9), (4096, 1, 65), (4097, 64, 65),
                                             (16384, 512, 70), (16387, 3, 1), (16384, 128, 300)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_coarse_takes_the_closest_centroids(nlist, nprobe, nq, metric):
    """Probe lists against float64 at sizes on both sides of every sample size, with centroids that occur twice."""
    g = torch.Generator(device="cuda")
    g.manual_seed(nlist + nprobe)
    cent = torch.randn(nlist, 64, generator=g, device="cuda")
    cent[nlist // 2:nlist // 2 + nlist // 8] = cent[:nlist // 8]
    off = torch.arange(nlist + 1, dtype=torch.int64)
    vec = torch.randn(nlist, 64, generator=g, device="cuda").half()
    ix = _hr().IvfIndex(cent, off, vec, torch.arange(nlist, device="cuda"))
    q = torch.randn(nq, 64, generator=g, device="cuda")
    probe, _ = ix.coarse(q, nprobe, metric)
    key = _keys(q.double(), cent.double(), metric)
    best = torch.topk(key, nprobe, dim=1).values
    got = key.gather(1, probe.long())
    # float32 sums of 64 products of values near 1, the norms among them: a few 2^-24 of |q|^2 + |x|^2 (below 400)
    assert float((got - best).abs().max()) < 4e-5
    assert all(len(set(p)) == nprobe for p in probe.cpu().tolist())
    # equal centroids: the lower index first (equal scores may be keys that |q|^2 - key rounds to the same value)
    p = probe.cpu().numpy()
    twin = (np.abs(p[:, 1:] - p[:, :-1]) == nlist // 2) & (np.minimum(p[:, 1:], p[:, :-1]) < nlist // 8)
    assert np.all(p[:, 1:][twin] > p[:, :-1][twin])
    ix.close()
