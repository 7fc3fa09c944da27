"""All-pairs MRCA kernels at the edges of their workgroups (1,024 columns, one to
eight rows) against the oracle on a sample of the surfaces, with counters from
0 to the top of the 32-bit range; outputs of pairs outside the matrix are not
touched."""
import ctypes

import numpy as np
import pytest

import oracle
from gpu_helpers import say
from paper_2405_03605_amd import load

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("sites,bits,policy", [(32, 1, 0), (16, 4, 0), (32, 1, 1), (64, 1, 1),
                                               (32, 2, 1), (64, 1, 2)])
@pytest.mark.parametrize("n,kc", [(255, 5), (1024, 1), (1025, 3), (2500, 5), (3073, 40)])
def test_matrix_edges(sites, bits, policy, n, kc):
    import torch
    say(f"mrca n={n} kc={kc} sites={sites} bits={bits} policy={policy}")
    words = sites * bits // 32
    rng = np.random.default_rng(n + 7 * policy + sites)
    T = np.where(rng.random(n) < 0.5, rng.integers(0, 1 << 32, n), 70000 + rng.integers(0, 90, n))
    T[:4] = (0, 1, (1 << 32) - 1, 1 << 31)
    T = T.astype(np.uint32)
    D = rng.integers(0, 1 << 32, (n, words), dtype=np.uint64).astype(np.uint32)
    related = rng.random(n) < 0.5
    D[related] = D[0] ^ (D[related] & rng.integers(0, 1 << 32, (int(related.sum()), words),
                                                   dtype=np.uint64).astype(np.uint32) & 0x11010101)
    lib, dev = load(), "cuda:0"
    t, d = (torch.from_numpy(a.view(np.int32).copy()).to(dev) for a in (T, D))
    ws = torch.empty(int(lib.ga_mrca_workspace_bytes(n)), dtype=torch.uint8, device=dev)
    guard = 4096
    out = torch.full((2, n * n + guard), -7, dtype=torch.int32, device=dev)
    p = lambda x: ctypes.c_void_p(x.data_ptr())  # noqa: E731
    code = lib.ga_mrca_matrix_ex(p(t), p(d), n, sites, bits, policy, kc,
                                 p(ws) if policy == 0 else None, ws.numel() if policy == 0 else 0,
                                 p(out[0]), p(out[1]),
                                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert code == 0
    torch.cuda.synchronize()
    assert bool((out[:, n * n:] == -7).all())
    L, U = (out[i, :n * n].cpu().numpy().view(np.uint32).reshape(n, n) for i in (0, 1))
    pick = np.unique(np.concatenate([[0, 1, 2, 3, n - 2, n - 1], rng.integers(0, n, 120)]))
    L0, U0 = oracle.mrca_interval_matrix(T[pick], D[pick], sites, kc, bits, policy=policy)
    assert np.array_equal(U[np.ix_(pick, pick)], U0)
    assert np.array_equal(L[np.ix_(pick, pick)], L0)
