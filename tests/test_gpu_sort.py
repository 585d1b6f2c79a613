"""The training step's and APAN's stable sort by node at the edges of its
tiles (2,048 keys) and digits: fewer keys than a tile, a tile exactly, one
more, node ids of one bit and of many, every contributor on one node.  A wrong
place in the sort shows in the gradients and mailboxes, which the oracle gives
(tolerances of tests/test_gpu_train.py and tests/test_gpu_apan.py)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import custom_workload, make_predictor, make_weights  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2402_15113_amd import tgm
    tgm.lib()


def stream(N, E, B, nb, seed=0, hub=False):
    r = np.random.default_rng(seed)
    src, dst, neg = (r.integers(0, N, E) for _ in range(3))
    if hub:
        src[:], neg[:] = 0, 0
    t = np.sort(r.integers(0, max(E // 3, 2), E)).astype(np.float64)
    f = r.standard_normal((E, 4)).astype(np.float32)
    return custom_workload(f"sort{N}_{B}", N, src, dst, t, neg, f, M=8, D_t=6, H=2, nb=nb, B=B,
                           s=1, seed=seed)


# contributors of a batch: 3 B (nb + 1); deliveries: 2 B (nb + 1)
@pytest.mark.parametrize("N,B,nb,hub", [(2, 5, 3, False), (700, 62, 10, False),
                                        (256, 256, 3, False), (255, 512, 3, False),
                                        (3000, 171, 3, False), (1025, 1025, 4, True),
                                        (40_000, 700, 2, False)])
def test_gradients_and_mailboxes(orc, N, B, nb, hub):
    from test_gpu_apan import apan_pair
    from test_gpu_train import train_pair
    wl = stream(N, 4 * B, B, nb, hub=hub)
    print(f"[sort] N={N} B={B} nb={nb} hub={hub}", flush=True)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random")
    train_pair(orc, wl, w, make_predictor(wl.M, seed=5), wl.n_iters, s=1, lr=1e-3)
    wa = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random", model="apan", K_mb=4)
    apan_pair(orc, wl, wa, wl.n_iters)
