"""The grouped GEMM of the training step and of APAN at the edges of its
tiles, against the fp64 oracle: widths around 4 (its vectors), 64 and 112 (its
tiles) and 32 (its steps), odd leading dimensions, every tile height (chosen
by the batch), heads narrower than a vector, and reductions from a few rows to
several parts.  Tolerances: the training tests' (tests/test_gpu_train.py)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import make_predictor, make_weights  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2402_15113_amd import tgm
    tgm.lib()


@pytest.mark.parametrize("M,H,D_e,D_t,B,nb", [
    (2, 1, 0, 1, 3, 4),        # narrower than a vector, no whole step
    (6, 3, 3, 5, 7, 10),       # two-wide heads
    (33, 1, 31, 32, 40, 10),   # one past a step
    (64, 2, 1, 63, 150, 5),    # whole tiles, two-part rows
    (112, 4, 190, 64, 90, 12), # 112-wide tiles, more slots than a wavefront keeps
    (116, 2, 201, 130, 25, 3), # one vector past them; the wide slot rows
    (100, 25, 40, 20, 500, 10),  # heads of 4; several parts of a reduction
])
def test_training_products_at_tile_edges(orc, M, H, D_e, D_t, B, nb):
    from test_gpu_parity import tie_heavy
    from test_gpu_train import train_pair
    wl = tie_heavy(11, N=13 + B // 2, E=6 * B, M=M, H=H, D_e=D_e, D_t=D_t, B=B, nb=nb)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=6, beta="random")
    print(f"[gemm] M={M} H={H} D_e={D_e} D_t={D_t} B={B} nb={nb}", flush=True)
    train_pair(orc, wl, w, make_predictor(wl.M, seed=3), wl.n_iters, s=wl.s, lr=1e-3)


def test_infinite_weights_in_the_overlapped_step(orc):
    """A reduction's last step of 32 overlaps the one before where its length
    is no multiple of 32 (62: elements 30 and 31 are in both).  An infinite
    weight there, of an update gate and an edge feature, saturates the gate; it
    is no NaN."""
    import numpy as np

    from test_gpu_apan import apan_pair
    from test_gpu_parity import tie_heavy
    wl = tie_heavy(7, N=30, E=200, M=8, H=1, D_e=40, D_t=6, B=20, nb=4)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random", model="apan", K_mb=4)
    W = np.array(w.W_ih, dtype=np.float32)   # [3 M x 62]: mail (16 + 40), time codes
    W[wl.M + 1, 30], W[wl.M + 3, 31] = np.inf, -np.inf
    w.W_ih = W
    apan_pair(orc, wl, w, wl.n_iters)
