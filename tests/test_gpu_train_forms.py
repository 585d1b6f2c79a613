"""The training attention's two forms at the edges of their ranges, against the
fp64 oracle: rows of up to 384 time codes stay in a wavefront's registers and
the products run over (root, head) rows; wider ones take the products over
slots, and so do 8 heads or more whose rows are loaded again for each head
(more than 10 slots, or 5 of wide rows) and 32 or more whose rows are not.  Also the wide rows (more than 192 edge features) with more slots than
they keep at a time, whose heads' sums go through memory.  Tolerances: the
training tests' (tests/test_gpu_train.py)."""
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


def pair(orc, M, H, D_e, D_t, B, nb):
    from test_gpu_parity import tie_heavy
    from test_gpu_train import train_pair
    wl = tie_heavy(12, N=13 + B // 2, E=6 * B, M=M, H=H, D_e=D_e, D_t=D_t, B=B, nb=nb)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=6, beta="random")
    print(f"[forms] M={M} H={H} D_e={D_e} D_t={D_t} B={B} nb={nb}", flush=True)
    train_pair(orc, wl, w, make_predictor(wl.M, seed=3), wl.n_iters, s=wl.s, lr=1e-3)


@pytest.mark.parametrize("M,H,D_e,D_t,B,nb", [
    (32, 2, 0, 383, 20, 10), (32, 2, 0, 384, 20, 10), (32, 2, 0, 385, 20, 10),
    (100, 2, 0, 416, 30, 10), (20, 5, 7, 430, 12, 33), (33, 1, 1, 500, 9, 48)])
def test_time_code_widths(orc, M, H, D_e, D_t, B, nb):
    pair(orc, M, H, D_e, D_t, B, nb)


@pytest.mark.parametrize("M,H,D_e,D_t,B,nb", [
    (36, 3, 193, 33, 20, 6), (128, 4, 256, 20, 15, 17), (64, 2, 200, 140, 20, 64)])
def test_wide_rows_in_parts(orc, M, H, D_e, D_t, B, nb):
    pair(orc, M, H, D_e, D_t, B, nb)


@pytest.mark.parametrize("M,H,D_e,D_t,B,nb", [
    (14, 7, 5, 9, 25, 11), (16, 8, 5, 9, 25, 11), (16, 8, 5, 9, 25, 10), (64, 8, 17, 129, 25, 5),
    (64, 8, 17, 129, 25, 6), (62, 31, 8, 16, 25, 10), (64, 32, 8, 16, 25, 10),
    (48, 48, 0, 8, 40, 10), (120, 24, 30, 40, 30, 64), (32, 8, 0, 4, 200, 20)])
def test_head_counts(orc, M, H, D_e, D_t, B, nb):
    pair(orc, M, H, D_e, D_t, B, nb)
