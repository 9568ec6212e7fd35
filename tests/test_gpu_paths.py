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


# rows over many board contexts: short sequences stay carried, those of many
# or large groups are cut; a captured product carries
CUT_CASES = [
    ("carried", lambda: I.small_turn_river(1, deck_size=9, n_board=3, cards_per_hand=2, bet_fracs=(0.5,),
                                           max_raises=0, stack=8.0)),
    ("carried_8", lambda: I.small_turn_river(2, deck_size=9, n_board=2, bet_fracs=(0.5, 1.0))),
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


# FP64 best responses on pieces of the treeplex: one piece, pieces under
# pieces, treeplex roots beside pieces that hang from a parent, whole
# treeplexes beyond 64 rows, one hand, more than eight actions
GAP_CASES = [
    ("tiny", lambda: I.tiny_config(), (64, 8)),
    ("river_roots", lambda: I.river_config(seed=3, n_keep=(17, 65), bet_fracs=(0.33, 0.75, 1.5), max_raises=4,
                                           stack=900.0), (64, 8, 13)),
    ("whole_menu", lambda: I.libratus_river(seed=2, n_keep=(33, 16), stack=900.0), (None, 64, 9)),
    ("many_actions", lambda: I.river_config(seed=5, n_keep=(40, 1), stack=20000.0, max_raises=1,
                                            bet_fracs=tuple(0.1 * k for k in range(1, 13))), (None, 64, 16)),
    ("turn_2card", lambda: I.small_turn_river(3, deck_size=13, n_board=3, cards_per_hand=2, bet_fracs=(0.5, 1.0),
                                              max_raises=1, stack=30.0, zero_frac=0.2), (64, 8)),
]


@pytest.mark.parametrize("name,fn,cuts", GAP_CASES, ids=[c[0] for c in GAP_CASES])
def test_best_responses_on_pieces(name, fn, cuts):
    d = fn()
    g = _game([d, I.small_river(0)])
    rng = np.random.default_rng(9)
    plans = [[], []]
    for i in range(2):
        for p in range(2):
            L = g.layouts[i][p]
            v = rng.random((L["n_seq"], L["n_hands"])) + 0.01
            for parent, first, n in zip(L["infoset_parent"], L["infoset_first"], L["infoset_nact"]):
                v[first:first + n] /= v[first:first + n].sum(axis=0)
                if parent >= 0:
                    v[first:first + n] *= v[parent]
            plans[p].append(v)
    x, y = (torch.from_numpy(g.pack(p, plans[p], dtype=np.float64)).cuda() for p in range(2))
    refs = [solver.saddle_gap(payoff.Game(di), plans[0][i], plans[1][i]) for i, di in enumerate((d, I.small_river(0)))]
    for cut in cuts:
        if cut is not None:
            g.solver_set_task_rows(cut)
        got = g.saddle_gap_of(x, y)
        for i, di in enumerate((d, I.small_river(0))):
            for k in range(3):
                assert abs(got[k][i] - refs[i][k]) <= 1e-9 * 2 * di.contrib, (cut, i, k, got[k][i], refs[i][k])


# the network's inference kernel: single rows, remainders of 32- and 128-row
# tiles, both sides of the row count where the tile changes, more tiles than
# workgroups
@pytest.mark.parametrize("rows", [1, 31, 32, 33, 1000, 8191, 8192, 8193, 32769, 66001])
def test_network_inference(rows):
    _game(I.tiny_config()).close()
    from paper_2112_03804_amd import warmstart
    gen = torch.Generator(device="cuda").manual_seed(rows)
    net = warmstart.WarmMLP(seed=rows)
    for k in ("b1", "b2", "b3"):
        net.p[k].copy_(0.2 * torch.randn(net.p[k].shape, generator=gen, device="cuda"))
    X = torch.randn((rows + 3, warmstart.D_IN), generator=gen, device="cuda").to(torch.bfloat16)
    got = net.logits(X[1:], rows)
    # the layer-by-layer path rounds the same activations to BF16, so the two
    # differ by FP32 summation order (512 terms: 512 * 2^-24 of the summed
    # magnitudes) and by the rare activation that it rounds the other way
    # (2^-8 of one term)
    ref = net.forward(X[1:], rows).clone()
    w3 = net.pb["W3"].float().abs()
    h2 = net._ws["H2b"][:rows].float().abs()
    mag = h2 @ w3.t().contiguous() + net.p["b3"].abs()
    top = (h2.max(dim=1, keepdim=True).values * w3.max(dim=1).values[None, :])
    assert got.shape == (rows, warmstart.K)
    assert ((got - ref).abs() <= 512 * 2.0 ** -24 * mag + 2 * 2.0 ** -8 * top).all()
    # and nearly all of them by the summation order alone
    assert ((got - ref).abs() <= 512 * 2.0 ** -24 * mag).float().mean() > 0.98


# FP64 products: both sides of every hands-per-thread class and of the 512
# threads of a workgroup, one hand, one-card hands, several items per chunk
F64_CASES = ([("n%d_%d" % n, lambda n=n: I.river_config(seed=n[0], n_keep=n, bet_fracs=(0.5,), max_raises=0))
              for n in [(1, 1081), (2, 1), (255, 256), (257, 512), (513, 511), (768, 769), (1024, 1025), (1081, 1023)]]
             + [("cards1", lambda: I.small_river(2, deck_size=40, cards_per_hand=1)),
                ("runouts", lambda: I.small_turn_river(6, deck_size=16, n_board=3, cards_per_hand=2, stack=12.0,
                                                       zero_frac=0.2))])


@pytest.mark.parametrize("name,fn", F64_CASES, ids=[c[0] for c in F64_CASES])
def test_fp64_products(name, fn):
    d = fn()
    g = _game([d, I.small_river(0)])
    per, (x, y) = _vectors(g, 11, np.float64)
    Ay, ATx = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
    g.matvec_A_f64(y, Ay)
    g.matvec_AT_f64(x, ATx)
    got_A, got_AT = g.unpack(0, Ay.cpu().numpy()), g.unpack(1, ATx.cpu().numpy())
    for i, di in enumerate((d, I.small_river(0))):
        o = payoff.Game(di)
        xi, yi = per[0][i], per[1][i]
        lim_A = 1e-12 * payoff.abs_matvec_A(o, yi) + 1e-15 * o.abs_row_sums().max() * yi.max()
        lim_AT = 1e-12 * payoff.abs_matvec_AT(o, xi) + 1e-15 * o.abs_col_sums().max() * xi.max()
        assert (np.abs(got_A[i] - o.matvec_A(yi)) <= lim_A).all()
        assert (np.abs(got_AT[i] - o.matvec_AT(xi)) <= lim_AT).all()
    # padding is written as 0
    for p, v in ((0, Ay), (1, ATx)):
        flat = v.cpu().numpy()
        for L in (l[p] for l in g.layouts):
            rows = flat[L["vec_offset"]:L["vec_offset"] + L["n_seq"] * L["stride"]].reshape(L["n_seq"], L["stride"])
            assert (rows[:, L["n_hands"]:] == 0).all()


# running averages over segments of iterations: any split of the same
# iterations into calls gives the same bits, captured or not, with retired
# instances, for every weight power
AVG_CASES = [
    ("tiny", lambda: [I.tiny_config()], dict(kind="rm+")),
    ("batch", lambda: I.batched_configs(3, seed=8, n_lo=40, n_hi=300), dict(kind="dcfr", gamma=3)),
    ("long_segments", lambda: [I.river_config(seed=4, n_keep=(211, 97), max_raises=2)], dict(kind="dcfr", gamma=2)),
    ("short_segments", lambda: [I.river_config(seed=6, bet_fracs=(0.33, 0.5, 1.0, 2.0), max_raises=4, stack=900.0)],
     dict(kind="rm+")),
]


@pytest.mark.parametrize("name,fn,rule", AVG_CASES, ids=[c[0] for c in AVG_CASES])
def test_averages_do_not_depend_on_the_split(name, fn, rule):
    descs = fn()
    states = []
    for split in ([1] * 41, [41], [8, 33], [7, 9, 25], [32, 8, 1]):
        g = _game(descs)
        g.solver_set_params(**rule)
        done = 0
        for n in split:
            g.solver_step(n)
            done += n
        if len(descs) > 1:
            g.solver_set_active([1, 0, 1])
            g.solver_step(10)
        torch.cuda.synchronize()
        states.append([g.solver_get_state(p) for p in range(2)] + [g.solver_get_weights()])
        g.close()
    for st in states[1:]:
        for p in range(2):
            for k in ("regret", "plan", "avg_sum"):
                assert np.array_equal(st[p][k], states[0][p][k]), (p, k)
            assert (st[p]["t"], st[p]["wsum"]) == (states[0][p]["t"], states[0][p]["wsum"])
        assert np.array_equal(st[2], states[0][2])


# a product's queries dealt to several workgroups per chunk (few chunks) and
# not (many copies of the game; a few share what CUs there are): the same bits,
# one to five hands per thread, own and opponent hand counts on either side of a
# thread's
@pytest.mark.parametrize("n_keep", [(257, 512), (513, 300), (700, 769), (1000, 1025), (1081, 1081), (256, 1030)])
def test_sliced_queries(n_keep):
    d = I.river_config(seed=31, n_keep=n_keep, bet_fracs=(0.5, 1.0), max_raises=2, stack=30.0)
    res = []
    for copies in (1, 5, 9, 70):
        g = _game([d] * copies)
        rng = np.random.default_rng(3)
        one = [rng.random((g.layouts[0][p]["n_seq"], g.layouts[0][p]["n_hands"])).astype(np.float32) for p in range(2)]
        x, y = (torch.from_numpy(g.pack(p, [one[p]] * copies, dtype=np.float32)).cuda() for p in range(2))
        Ay, ATx = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
        g.matvec_A(y, Ay)
        g.matvec_AT(x, ATx)
        By, BTx = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
        g.matvec_pair(y, x, By, BTx)
        torch.cuda.synchronize()
        for u, v in ((Ay, By), (ATx, BTx)):
            u, v = (t.cpu().numpy().reshape(copies, -1) for t in (u, v))
            assert np.array_equal(u, v) and (u == u[0]).all()
            res.append(u[0])
        g.close()
    for k in range(2, 8, 2):
        assert np.array_equal(res[0], res[k]) and np.array_equal(res[1], res[k + 1])


# the FP64 products don't depend on the schedules tried before the chosen one
@pytest.mark.parametrize("tried", [(), ((3, 8),), ((2, 1), (3, 64))])
@pytest.mark.parametrize("name,fn", CUT_CASES[1:3], ids=[c[0] for c in CUT_CASES[1:3]])
def test_fp64_products_after_tuning(name, fn, tried):
    d = fn()
    g, h = _game(d), _game(d)
    for k, r in tried:
        g.game_tune(k, r)
    g.game_tune(4, 2)
    _, (x, y) = _vectors(g, 6, np.float64)
    outs = []
    for q in (g, h):
        Ay, ATx = torch.full_like(x, 7.0), torch.full_like(y, 7.0)
        q.matvec_A_f64(y, Ay)
        q.matvec_AT_f64(x, ATx)
        torch.cuda.synchronize()
        outs.append((Ay.cpu().numpy(), ATx.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    g.close()
    h.close()


# regret updates' blocks in the order of the XCDs: copies of one game, so that
# launches have fewer blocks than a run, whole runs and a remainder; every copy
# gives the same bits, in pieces of one and of two depths
@pytest.mark.parametrize("copies", [2, 16, 37])
@pytest.mark.parametrize("rows", [16, 64])
def test_update_blocks_cover_every_copy(copies, rows):
    d = I.river_config(seed=9, n_keep=(150, 61), max_raises=2)
    g = _game([d] * copies)
    g.solver_set_rm_quad(0)
    g.solver_set_task_rows(rows)
    g.solver_step(6)
    torch.cuda.synchronize()
    for p in range(2):
        st = g.solver_get_state(p)
        for k in ("regret", "plan", "avg_sum"):
            v = st[k].reshape(copies, -1)
            assert np.abs(v[0]).max() > 0
            assert (v == v[0]).all(), (p, k)


# four lanes per hand: infosets of up to 4, 5 to 8 and more actions (one, two
# and more per lane), whole and in pieces; a step from random regrets against
# the oracle, the plan as the realization of the device's own regrets
@pytest.mark.parametrize("kind", ["rm+", "dcfr"])
@pytest.mark.parametrize("rows", [16, 64])
@pytest.mark.parametrize("sizes,raises", [(1, 2), (2, 2), (3, 2), (5, 1), (7, 1), (11, 1)])
def test_update_by_action_count(sizes, raises, rows, kind):
    d = I.river_config(seed=12, n_keep=(37, 21), bet_fracs=tuple(0.25 * (i + 1) for i in range(sizes)),
                       max_raises=raises, stack=500.0)
    o = payoff.Game(d)
    g = _game(d)
    if rows < 64:
        g.solver_set_task_rows(rows)
    g.solver_set_params(kind)
    rng = np.random.default_rng(sizes)
    ref = solver.RMPlus(o, kind=kind)
    for p in range(2):
        R = ((rng.random((o.S[p], o.N[p])) - 0.2) * 3.0).astype(np.float32).astype(np.float64)
        if kind == "rm+":
            R = np.maximum(R, 0.0)
        x = ref.tp[p].realization(ref.tp[p].behaviour_from_regret(R)).astype(np.float32).astype(np.float64)
        ref.R[p], ref.x[p] = R, x
        ref.sum[p] = np.zeros_like(x)
        g.solver_set_state(p, regret=g.pack(p, [R]), plan=g.pack(p, [x]),
                           avg_sum=g.pack(p, [ref.sum[p]], np.float64), t=4, wsum=10.0)
    ref.t, ref.wsum = 4, 10.0
    g.solver_step(1)
    torch.cuda.synchronize()
    ref.step()
    for p in range(2):
        st = g.solver_get_state(p)
        R, x = g.unpack(p, st["regret"])[0], g.unpack(p, st["plan"])[0]
        assert np.abs(R - ref.R[p]).max() <= 1e-5 * max(1.0, np.abs(ref.R[p]).max()), p
        tp = ref.tp[p]
        assert np.abs(x - tp.realization(tp.behaviour_from_regret(R))).max() <= 1e-5, p
    g.close()


# a training step's kernels against the layer-by-layer path: remainders of the
# 32-row blocks and the 256-row losses, one split and many, with and without
# weights
@pytest.mark.parametrize("rows", [1, 31, 32, 33, 255, 257, 1000, 4097, 8192])
def test_training_gradients(rows):
    _game(I.tiny_config()).close()
    from paper_2112_03804_amd import warmstart
    gen = torch.Generator(device="cuda").manual_seed(rows)
    net = warmstart.WarmMLP(seed=rows)
    for k in ("b1", "b2", "b3"):
        net.p[k].copy_(0.2 * torch.randn(net.p[k].shape, generator=gen, device="cuda"))
    # one spare element in front: the copy at an odd offset goes layer by layer
    buf = torch.randn((rows * warmstart.D_IN + 8,), generator=gen, device="cuda").to(torch.bfloat16)
    X = buf[:rows * warmstart.D_IN].view(rows, -1)
    shifted = torch.empty_like(buf)
    Xs = shifted[1:1 + rows * warmstart.D_IN].view(rows, -1)
    Xs.copy_(X)
    T = torch.rand((rows, warmstart.K), generator=gen, device="cuda")
    valid = torch.arange(warmstart.K, device="cuda")[None, :] < torch.randint(1, 9, (rows, 1), generator=gen, device="cuda")
    T = torch.where(valid, T / (T * valid).sum(dim=1, keepdim=True), torch.full_like(T, -1.0)).contiguous()
    W = torch.rand((rows,), generator=gen, device="cuda") if rows % 2 else None
    ref_loss = net.loss_and_grad(Xs, T, W, rows).clone()
    ref = {k: v.clone() for k, v in net.g.items()}
    ws = net._ws
    mag = {"W3": (ws["dZ3b"], ws["H2b"]), "W2": (ws["dZ2b"], ws["H1b"]), "W1": (ws["dZ1b"], X)}
    cols = {"b3": ws["dZ3"], "b2": ws["dZ2"], "b1": ws["dZ1"]}
    for v in net.g.values():
        v.fill_(7.0)
    loss = net.loss_and_grad(X, T, W, rows)
    assert loss.shape == ref_loss.shape
    assert ((loss - ref_loss).abs() <= 1e-4 * ref_loss.abs()).all()
    # the same values are rounded to BF16 on both paths after FP32 sums in
    # another order: a value may round the other way (2^-8 of it) at each of
    # the layers before it, which bounds every term of a gradient
    for k, (d, h) in mag.items():
        lim = d[:rows].float().abs().t().contiguous() @ h[:rows].float().abs()
        assert ((net.g[k] - ref[k]).abs() <= 4 * 2.0 ** -8 * lim + 1e-30).all(), k
    for k, d in cols.items():
        assert ((net.g[k] - ref[k]).abs() <= 4 * 2.0 ** -8 * d[:rows].abs().sum(dim=0) + 1e-30).all(), k
    # and few do: the gradients agree far closer as a whole
    for k in ref:
        assert (net.g[k] - ref[k]).norm() <= 2e-3 * ref[k].norm(), k
