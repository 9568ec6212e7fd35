"""Paths of the dispatch against one another and the oracle, at the sizes where
a rule changes path (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

from paper_2112_03804_amd import instances as I
from oracle import payoff, solver

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _game(d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_03804_amd import pmx
    return pmx.Game(d)


def _vectors(g, seed, dtype):
    """Random plans of both players (rows padded with 0)."""
    rng = np.random.default_rng(seed)
    per = [[rng.random((L[p]["n_seq"], L[p]["n_hands"])).astype(dtype) for L in g.layouts] for p in range(2)]
    return per, [torch.from_numpy(g.pack(p, per[p], dtype=dtype)).cuda() for p in range(2)]


# rows over many board contexts: a small turn game's sequences stay carried
# (fewer than eight groups), longer ones are cut; a captured product carries
CUT_CASES = [
    ("carried", lambda: I.small_turn_river(1, deck_size=9, n_board=3, cards_per_hand=2, bet_fracs=(0.5,),
                                           max_raises=0, stack=8.0)),
    ("cut_at_8", lambda: I.small_turn_river(2, deck_size=9, n_board=2, bet_fracs=(0.5, 1.0))),
    ("cut_20", lambda: I.small_turn_river(3, deck_size=23, n_board=3, cards_per_hand=2, bet_fracs=(0.5,),
                                          max_raises=1, stack=12.0, zero_frac=0.2)),
    ("cut_two_classes", lambda: [I.small_turn_river(4, deck_size=14, n_board=3, cards_per_hand=2, stack=9.0),
                                 I.small_turn_river(5, deck_size=30, n_board=4, cards_per_hand=2, stack=9.0),
                                 I.small_river(0)]),
]


@pytest.mark.parametrize("name,fn", CUT_CASES, ids=[c[0] for c in CUT_CASES])
def test_cut_rows_equal_carried_rows(name, fn):
    d = fn()
    g = _game(d)
    descs = d if isinstance(d, list) else [d]
    per, (x, y) = _vectors(g, 5, np.float32)
    Ay, ATx = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
    g.matvec_pair(y, x, Ay, ATx)
    Ay1, ATx1 = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
    g.matvec_A(y, Ay1)
    g.matvec_AT(x, ATx1)
    torch.cuda.synchronize()
    # a captured product takes the carrying kernel: the same bits, on every replay
    Ac, Tc = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.matvec_A(y, Ac)
        g.matvec_AT(x, Tc)
    for _ in range(3):
        Ac.fill_(7.0)
        Tc.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        for got in ((Ay, ATx), (Ay1, ATx1)):
            assert torch.equal(got[0], Ac) and torch.equal(got[1], Tc)
    got_A, got_AT = g.unpack(0, Ay.cpu().numpy()), g.unpack(1, ATx.cpu().numpy())
    for i, di in enumerate(descs):
        o = payoff.Game(di)
        xi, yi = per[0][i].astype(np.float64), per[1][i].astype(np.float64)
        lim_A = 1e-6 * payoff.abs_matvec_A(o, yi) + 1e-7 * o.abs_row_sums().max() * yi.max()
        lim_AT = 1e-6 * payoff.abs_matvec_AT(o, xi) + 1e-7 * o.abs_col_sums().max() * xi.max()
        assert (np.abs(got_A[i] - o.matvec_A(yi)) <= lim_A).all()
        assert (np.abs(got_AT[i] - o.matvec_AT(xi)) <= lim_AT).all()
