"""The attention by aggregation at the edges of its slot-row registers: edge
feature widths around 64, 128, 192 (where the packed rows take over) and 256,
time codes around 64 and 128, slot counts around 4, 10 and 16, one to four
heads (pairs of heads share a pass), against the fp64 oracle (tolerances of
tests/test_gpu_parity.py)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import make_weights  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2402_15113_amd import tgm
    tgm.lib()


@pytest.mark.parametrize("M,H,D_e,D_t,nb", [
    (4, 1, 1, 0, 1), (12, 3, 64, 64, 4), (16, 4, 65, 63, 5), (100, 2, 192, 128, 10),
    (20, 1, 193, 127, 9), (64, 2, 256, 64, 10), (112, 4, 256, 1, 16), (96, 3, 0, 128, 11),
    (36, 2, 127, 65, 15), (100, 4, 191, 100, 16), (32, 2, 193, 100, 4), (16, 1, 255, 65, 3),
    (100, 2, 256, 0, 10), (96, 3, 193, 63, 16), (8, 2, 200, 120, 1)])
def test_attention_rows(orc, M, H, D_e, D_t, nb):
    from test_gpu_parity import run_pair, tie_heavy
    wl = tie_heavy(5, N=40, E=400, M=M, H=H, D_e=D_e, D_t=D_t, B=37, nb=nb)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=7, beta="random")
    print(f"[attention] M={M} H={H} D_e={D_e} D_t={D_t} nb={nb}", flush=True)
    run_pair(orc, wl, w)
