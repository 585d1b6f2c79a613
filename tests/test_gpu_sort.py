"""The training step's and APAN's stable sort by node at the edges of its
tiles (2,048 keys) and digits: fewer keys than a tile, a tile exactly, one
more, more tiles than a scatter reads at a time (16), node ids of one bit and
of many, every contributor on one node; and the library sort that takes over
past 2^19 keys or 20 bits, on both sides of the line.  A wrong
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
                                        (40_000, 700, 2, False), (3000, 900, 12, False),
                                        (900, 1500, 8, True)])
def test_gradients_and_mailboxes(orc, N, B, nb, hub):
    from test_gpu_apan import apan_pair
    from test_gpu_train import train_pair
    wl = stream(N, 4 * B, B, nb, hub=hub)
    print(f"[sort] N={N} B={B} nb={nb} hub={hub}", flush=True)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random")
    train_pair(orc, wl, w, make_predictor(wl.M, seed=5), wl.n_iters, s=1, lr=1e-3)
    wa = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random", model="apan", K_mb=4)
    apan_pair(orc, wl, wa, wl.n_iters)


def test_gradients_around_the_library_sort(orc):
    """Batches of 524,355, 524,355 and 523,965 contributors of one trainer (64
    slots: 195 a batch event): past the line, and a last one below it."""
    from test_gpu_train import train_pair
    B, nb = 2689, 64
    wl = stream(6000, 2 * B + 2687, B, nb)
    print(f"[sort] B={B} nb={nb}", flush=True)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random")
    train_pair(orc, wl, w, make_predictor(wl.M, seed=5), wl.n_iters, s=1, lr=1e-3)


def test_gradients_with_every_tile(orc):
    """524,160 contributors: all 256 tiles of the sort."""
    from test_gpu_train import train_pair
    wl = stream(6000, 2 * 2688, 2688, 64)
    print("[sort] B=2688 nb=64", flush=True)
    w = make_weights(wl.M, wl.D_e, wl.D_t, seed=2, beta="random")
    train_pair(orc, wl, w, make_predictor(wl.M, seed=5), wl.n_iters, s=1, lr=1e-3)


def test_mailboxes_of_wide_node_ids(orc):
    """Node ids of 21 bits (N = 2^20 + 7).  The library's own node set ends at
    2^19 ids, so the sample's is made here."""
    from paper_2402_15113_amd import tgm
    from paper_2402_15113_amd.stage import ApanStage
    from test_gpu_parity import close, exact
    N, B, nb, K, M = (1 << 20) + 7, 60, 3, 2, 4
    r = np.random.default_rng(4)
    ids = np.unique(np.concatenate([np.arange(N - 9, N), np.arange(5), r.integers(0, N, 60)]))
    E = 5 * B + 11
    src, dst, neg = (r.choice(ids, E) for _ in range(3))
    t = np.sort(r.integers(0, 90, E)).astype(np.float64)
    f = r.standard_normal((E, 2)).astype(np.float32)
    wl = custom_workload("wide ids", N, src, dst, t, neg, f, M=M, D_t=3, H=1, nb=nb, B=B, s=1)
    w = make_weights(M, 2, 3, seed=3, beta="random", model="apan", K_mb=K)
    st, o = ApanStage(wl, w), orc.Oracle(wl, w)
    b, s = st.sb, st.stream
    for i in range(wl.n_iters):
        print(f"[sort] wide ids iter {i}", flush=True)
        lo = i * B
        n = min(B, E - lo)
        R = 3 * n
        tgm.tgm_batch_roots(st.g, lo, n, b.root, b.root_ts, stream=s)
        tgm.tgm_sample(st.g, b.root, b.root_ts, R, nb, b.nbr, b.eid, b.nts, b.cnt, stream=s)
        nbr = b.nbr[:R].long()
        on = nbr >= 0
        U = torch.unique(torch.cat([b.root[:R].long(), nbr[on]]))
        b.nodes[:U.numel()] = U.int()
        b.n_nodes.fill_(U.numel())
        b.root_pos[:R] = torch.searchsorted(U, b.root[:R].long()).int()
        b.nbr_pos[:R] = torch.where(on, torch.searchsorted(U, nbr), -1).int()
        tgm.tgm_apan_step(st.a, st.g, i, st._sbs, st.cap, st.mem_new, st.new_mem_ts, st.h,
                          stream=s)
        st.last = (i, n)
        g, q = st.outputs(), o.step()
        exact("U", g["U"], q.U)
        exact("f_mb_cnt", g["f_mb_cnt"], q.f_mb_cnt)
        mask = np.arange(K)[None, :] < q.f_mb_cnt[:, None]
        exact("f_mb_ts", g["f_mb_ts"][mask], q.f_mb_ts[mask])
        close("f_mb", g["f_mb"][mask], q.f_mb[mask])
        close("s_new", g["s_new"], q.s_new)
        close("h", g["h"], q.h)
    st.close()
