"""Calls at the edges of what the entry points take."""
import time

import numpy as np
import pytest

from paper_2112_03804_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _game(d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_03804_amd import pmx
    return pmx.Game(d)


def _net(seed):
    _game(I.tiny_config()).close()
    from paper_2112_03804_amd import warmstart
    gen = torch.Generator(device="cuda").manual_seed(seed)
    net = warmstart.WarmMLP(seed=seed)
    for k in ("b1", "b2", "b3"):
        net.p[k].copy_(0.2 * torch.randn(net.p[k].shape, generator=gen, device="cuda"))
    return net, gen


# entries past a row's hands are ignored on input and written as 0 on output:
# a plan loaded with anything there leaves no trace in the averages
@pytest.mark.parametrize("steps", [1, 3, 40])
@pytest.mark.parametrize("kind", ["rm+", "dcfr"])
def test_padding_of_a_loaded_plan(kind, steps):
    descs = [I.river_config(seed=4, n_keep=(33, 21), max_raises=1), I.small_river(0)]
    clean, dirty = _game(descs), _game(descs)
    for g in (clean, dirty):
        g.solver_set_params(kind)
        g.solver_step(5)
    torch.cuda.synchronize()
    pads = []
    for p in range(2):
        pad = np.ones(clean.elems[p], bool)
        for L in (l[p] for l in clean.layouts):
            rows = pad[L["vec_offset"]:L["vec_offset"] + L["n_seq"] * L["stride"]].reshape(L["n_seq"], L["stride"])
            rows[:, :L["n_hands"]] = False
        assert pad.any()
        pads.append(pad)
        st = clean.solver_get_state(p)
        for g, fill in ((clean, 0.0), (dirty, np.nan)):
            plan = st["plan"].copy()
            plan[pad] = fill
            g.solver_set_state(p, regret=st["regret"], plan=plan, avg_sum=st["avg_sum"], t=5, wsum=st["wsum"])
    for g in (clean, dirty):
        g.solver_step(steps)
    torch.cuda.synchronize()
    for p in range(2):
        a, b = clean.get_average_strategy(p), dirty.get_average_strategy(p)
        assert (a[pads[p]] == 0).all() and np.array_equal(a, b)
        s, t = clean.solver_get_state(p), dirty.solver_get_state(p)
        for k in ("regret", "plan", "avg_sum"):
            assert np.array_equal(s[k][~pads[p]], t[k][~pads[p]]), (p, k)
    assert np.array_equal(clean.saddle_gap()[0], dirty.saddle_gap()[0])


# products of one game on two streams, with other inputs each and nothing
# between them that waits: rows over many board contexts go through buffers of
# the game's own.  FP32 on the grouped schedule (terms) and on both others
# (partial rows), FP64 (partial rows); beside a solver that runs on a third
# stream, and beside replays of captured products
TURN = [("one_class", lambda: I.small_turn_river(3, deck_size=23, n_board=3, cards_per_hand=2, bet_fracs=(0.5,),
                                                 max_raises=1, stack=12.0, zero_frac=0.2)),
        ("two_classes", lambda: [I.small_turn_river(4, deck_size=14, n_board=3, cards_per_hand=2, stack=9.0),
                                 I.small_turn_river(5, deck_size=30, n_board=4, cards_per_hand=2, stack=9.0)])]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("tune", [None, (2, 2), (3, 1)])
@pytest.mark.parametrize("name,fn", TURN, ids=[c[0] for c in TURN])
def test_products_on_several_streams(name, fn, tune, dtype):
    g, n = _game(fn()), 12
    if tune:
        g.game_tune(*tune)
    gen = torch.Generator(device="cuda").manual_seed(8)
    x, y = (torch.rand((n, g.elems[p]), generator=gen, device="cuda", dtype=dtype) for p in range(2))
    prods = (g.matvec_A_f64, g.matvec_AT_f64) if dtype == torch.float64 else (g.matvec_A, g.matvec_AT)
    ref = [torch.full_like(x, 7.0), torch.full_like(y, 7.0)]
    for i in range(n):
        prods[0](y[i], ref[0][i])
        prods[1](x[i], ref[1][i])
        torch.cuda.synchronize()
    # captured products: the caller's streams again may replay them beside others
    cap, graph = [torch.full_like(x[0], 7.0), torch.full_like(y[0], 7.0)], torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        prods[0](y[0], cap[0])
        prods[1](x[0], cap[1])
    streams = [torch.cuda.Stream() for _ in range(4)]
    out = [torch.full_like(x, 7.0), torch.full_like(y, 7.0)]
    torch.cuda.synchronize()
    for rounds in range(3):
        for v in out + cap:
            v.fill_(7.0)
        torch.cuda.synchronize()
        for i in range(n):
            with torch.cuda.stream(streams[i % 2]):
                prods[0](y[i], out[0][i])
                prods[1](x[i], out[1][i])
            if i % 4 == 1:
                with torch.cuda.stream(streams[2]):
                    g.solver_step(1)
                with torch.cuda.stream(streams[3]):
                    graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], ref[0]) and torch.equal(out[1], ref[1])
        # a captured product sums a row without cutting it: rounding of the
        # partial rows (FP32 on schedules 2 and 3), up to a sum's magnitude
        for got, want in zip(cap, ref):
            tol = 1e-13 if dtype == torch.float64 else 1e-6
            assert ((got - want[0]).abs() <= tol * want[0].abs().max()).all()
    # the solver's own products were not disturbed either
    h = _game(fn())
    if tune:
        h.game_tune(*tune)
    for _ in range(9):
        h.solver_step(1)
    torch.cuda.synchronize()
    for p in range(2):
        s, t = g.solver_get_state(p), h.solver_get_state(p)
        assert all(np.array_equal(s[k], t[k]) for k in ("regret", "plan", "avg_sum"))


# a batch of turn games with retired instances: the solver's lists of cut rows
# without them give what the instances give alone
@pytest.mark.parametrize("active", [[1, 0, 1, 0], [0, 0, 1, 0]])
def test_cut_rows_of_active_instances(active):
    descs = [I.small_turn_river(s, deck_size=20, n_board=3, cards_per_hand=2, stack=9.0) for s in range(4)]
    g = _game(descs)
    g.solver_step(6)
    g.solver_set_active(active)
    g.solver_step(40)
    torch.cuda.synchronize()
    for i, on in enumerate(active):
        h = _game([descs[i]] * 4)   # the same schedules: a batch of copies
        h.solver_step(46 if on else 6)
        torch.cuda.synchronize()
        for p in range(2):
            s, t = g.solver_get_state(p), h.solver_get_state(p)
            for k in ("regret", "plan", "avg_sum"):
                assert np.array_equal(g.unpack(p, s[k])[i], h.unpack(p, t[k])[0]), (i, p, k)
        h.close()


# no rows: an empty result, as a loop over no chunks gives
def test_inference_of_no_rows():
    net, _ = _net(1)
    from paper_2112_03804_amd import pmx, warmstart
    X = torch.empty((0, warmstart.D_IN), dtype=torch.bfloat16, device="cuda")
    out = net.logits(X, 0)
    assert out.shape == (0, warmstart.K) and out.dtype == torch.float32
    assert net.logits(torch.zeros((5, warmstart.D_IN), dtype=torch.bfloat16, device="cuda"), 0).shape[0] == 0
    # through the ABI: nothing to do, whatever the row pointers are
    d, p, pb = pmx.dptr, net.p, net.pb
    assert pmx.lib().mlp_forward_bf16(0, None, d(pb["W1"]), d(p["b1"]), d(pb["W2"]), d(p["b2"]), d(pb["W3"]),
                                      d(p["b3"]), None, None, pmx.stream_ptr()) == 0


# every parameter and gradient at an odd offset of one flat buffer, as
# programs that flatten their parameters keep them
@pytest.mark.parametrize("rows", [1, 77, 700])
@pytest.mark.parametrize("which", ["p", "pb", "g"])
def test_parameters_in_a_flat_buffer(which, rows):
    net, gen = _net(rows)
    from paper_2112_03804_amd import warmstart
    X = torch.randn((rows, warmstart.D_IN), generator=gen, device="cuda").to(torch.bfloat16)
    T = torch.rand((rows, warmstart.K), generator=gen, device="cuda")
    T = (T / T.sum(dim=1, keepdim=True)).contiguous()
    W = torch.rand((rows,), generator=gen, device="cuda")
    ref = net.forward(X, rows).clone()
    ref_loss = net.loss_and_grad(X, T, W, rows).clone()
    ref_g = {k: v.clone() for k, v in net.g.items()}
    d = getattr(net, which)
    flat = torch.empty(sum(v.numel() for v in d.values()) + 1, dtype=next(iter(d.values())).dtype, device="cuda")
    at = 1   # lengths are multiples of 8: every view starts one value past a 16-byte boundary
    for k, v in d.items():
        view = flat[at:at + v.numel()].view(v.shape)
        view.copy_(v)
        d[k] = view
        at += v.numel()
    assert all(v.data_ptr() % 16 for v in d.values())
    got = net.logits(X, rows)
    loss = net.loss_and_grad(X, T, W, rows)
    # the kernels of either path round the same values to BF16 and differ by
    # the order of FP32 sums, and by the rare value rounded the other way
    assert ((got - ref).norm() <= 2e-3 * ref.norm())
    assert ((loss - ref_loss).abs() <= 1e-4 * ref_loss.abs()).all()
    for k in ref_g:
        assert (net.g[k] - ref_g[k]).norm() <= 2e-3 * ref_g[k].norm(), k
    before = {k: v.clone() for k, v in net.p.items()}
    net.adam(lr=1e-3)
    assert all(not torch.equal(before[k], net.p[k]) for k in before)
    assert all(torch.equal(net.p[k].to(torch.bfloat16), net.pb[k]) for k in net.pb)


# the plans that the averages take together (28 bytes per element in segments
# of eight iterations) are allocated by the first solver step, as many as fit:
# a game that only just fits still solves, to the same bits
def test_solver_memory():
    descs = I.batched_configs(160, seed=2)
    g = _game(descs)
    free = lambda: torch.cuda.mem_get_info()[0]
    torch.cuda.synchronize()
    f0 = free()
    h = _game(descs)
    torch.cuda.synchronize()
    made = f0 - free()
    seg = 28 * sum(h.elems)
    assert seg > 200 << 20
    x, y = (torch.rand(n, device="cuda") for n in h.elems)
    Ay, ATx = torch.empty_like(x), torch.empty_like(y)
    f1 = free()
    h.matvec_pair(y, x, Ay, ATx)
    torch.cuda.synchronize()
    assert f1 - free() < seg // 4
    h.solver_step(40)
    torch.cuda.synchronize()
    assert f1 - free() > seg - (16 << 20)
    ref = [h.solver_get_state(p) for p in range(2)]
    h.close()
    g.close()
    torch.cuda.empty_cache()
    # room for a game and less than half of its segments
    room, hog = made + int(0.45 * seg), []
    for _ in range(10):   # memory given back may be counted late
        if free() > room + (8 << 20):
            hog.append(torch.empty(free() - room, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        time.sleep(0.05)
    print("left", free() >> 20, "MB, game", made >> 20, "MB, segments", seg >> 20, "MB", flush=True)
    if not room - seg // 8 < free() < room + seg // 8:
        pytest.skip("the memory left does not settle")
    g = _game(descs)
    before = free()
    g.solver_step(3)
    g.solver_step(37)
    torch.cuda.synchronize()
    assert before - free() < seg // 2
    for p in range(2):
        st = g.solver_get_state(p)
        assert all(np.array_equal(st[k], ref[p][k]) for k in ("regret", "plan", "avg_sum"))
    g.close()
    del hog
    torch.cuda.empty_cache()


# one iteration is two products and two updates: the averages take no launch of
# their own then (programs that step one iteration at a time)
@pytest.mark.parametrize("steps,launches", [(1, 4), (5, 21)])
def test_launches_of_a_step(steps, launches):
    import ctypes
    g = _game(I.tiny_config())
    g.solver_step(1)
    torch.cuda.synchronize()
    from paper_2112_03804_amd import pmx
    L, graph, n = pmx.lib(), ctypes.c_void_p(), ctypes.c_size_t()
    stream = torch.cuda.Stream()
    assert L.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.c_int(2)) == 0
    g.solver_step(steps, stream=stream.cuda_stream)
    assert L.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert L.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert L.hipGraphDestroy(graph) == 0
    assert n.value == launches
    g.close()


# weight gradients of long batches: sums over rows are cut into ranges, so that
# one row of large activations hides the others of its own range at most (a
# single FP32 sum would lose them all).  Row 0's second hidden activation is
# 2^30, the others' 1; the output gradients are 1/8; every product is exact,
# and 32 rows' 1s are less than half a unit (128) of 2^30's sum
@pytest.mark.parametrize("rows,rows_of_a_range", [(8192, 512), (32768, 1024), (65536, 1024), (262144, 4096)])
def test_sums_of_long_batches(rows, rows_of_a_range):
    net, _ = _net(3)
    from paper_2112_03804_amd import warmstart
    for k in net.p:
        net.p[k].zero_()
    for k in net.pb:
        net.pb[k].zero_()
    net.pb["W1"][5, 2] = 1.0
    net.pb["W2"][9, 5] = 1.0
    X = torch.zeros((rows, warmstart.D_IN), dtype=torch.bfloat16, device="cuda")
    X[:, 2] = 1.0
    X[0, 2] = 2.0 ** 30
    T = torch.zeros((rows, warmstart.K), device="cuda")
    T[:, 0] = 1.0
    loss = net.loss_and_grad(X, T, None, rows)
    # up to 20 partial sums more, each rounded to 128
    want = 0.125 * (2.0 ** 30 + rows - 1)
    assert abs(float(net.g["W3"][1, 9]) - want) <= 0.125 * (rows_of_a_range + 20 * 64)
    assert abs(float(net.g["b3"][1]) - 0.125 * rows) <= 1e-5 * rows
    # the loss of 256 rows is a sum in a tree of depth 8
    assert loss.shape == (rows // 256,)
    assert ((loss.double() - 256 * np.log(8.0)).abs() <= 256 * np.log(8.0) * 2.0 ** -24 * (8 + 8)).all()


# rows with non-finite values: the logits of the others are the same bits as
# without them, and where the layer-by-layer path gives a non-finite logit, so
# does the fused one (a warm start falls back row by row on these).  ReLU takes
# a NaN to 0 on either path, so that weights of both signs leave finite logits,
# and non-negative ones infinities in the rows of +inf and 3e38
@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("rows", [40, 300, 8192, 8500])
def test_non_finite_rows(rows, positive):
    net, gen = _net(rows)
    from paper_2112_03804_amd import warmstart
    if positive:
        for v in net.pb.values():
            v.abs_()
    X = torch.randn((rows, warmstart.D_IN), generator=gen, device="cuda").to(torch.bfloat16)
    T = torch.full((rows, warmstart.K), 1.0 / warmstart.K, device="cuda")
    bad = torch.zeros(rows, dtype=torch.bool, device="cuda")
    clean, clean_loss = net.logits(X, rows), net.loss_and_grad(X, T, None, rows).clone()
    for k, v in ((3, float("nan")), (17, float("inf")), (31, -float("inf")), (rows - 1, 3e38)):
        X[k] = v
        bad[k] = True
    got, ref = net.logits(X, rows), net.forward(X, rows)[:rows]
    assert torch.equal(got[~bad], clean[~bad])
    assert torch.equal(torch.isfinite(got), torch.isfinite(ref))
    if positive:
        assert not torch.isfinite(got[[17, rows - 1]]).any()
    loss = net.loss_and_grad(X, T, None, rows)
    hit = torch.zeros(((rows + 255) // 256) * 256, dtype=torch.bool, device="cuda")
    hit[:rows] = bad & ~torch.isfinite(ref).all(dim=1)
    hit = hit.view(-1, 256).any(dim=1)
    assert torch.equal(~torch.isfinite(loss), hit)
    clear = torch.ones_like(hit)
    clear[[0, (rows - 1) // 256]] = False
    assert torch.equal(loss[clear], clean_loss[clear])


# a first step that the caller captures: nothing is allocated then, and replays
# are iterations like any other
@pytest.mark.parametrize("steps", [1, 3, 9])
@pytest.mark.parametrize("fn", [I.tiny_config, lambda: I.batched_configs(3, seed=8, n_lo=40, n_hi=300)], ids=["tiny", "batch"])
def test_captured_first_step(fn, steps):
    g, h = _game(fn()), _game(fn())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.solver_step(steps)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        g.solver_step(2)
        h.solver_step(steps)
        h.solver_step(2)
        torch.cuda.synchronize()
        for p in range(2):
            s, t = g.solver_get_state(p), h.solver_get_state(p)
            assert all(np.array_equal(s[k], t[k]) for k in ("regret", "plan", "avg_sum"))
    g.close()
    h.close()
