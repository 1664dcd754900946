"""GPU tests of the request loop (include/bgserve.h) through the C ABI: the
device generator against the Philox oracle bit for bit, final client states
against the CPU replay, results identical alone and in the mix, the timing
outputs and the memory budget."""
import numpy as np
import pytest
import torch

from oracle import philox, serving
from paper_2203_09353_amd import bgemm, serve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    hd = bgemm.Handle()
    yield hd
    hd.close()


@pytest.mark.parametrize("n,client,j", [(1, 0, 0), (5, 3, 7), (32, 63, 2 ** 40 + 3), (33, 1, 12),
                                        (128, 2, 0), (257, 9, 1)])
def test_generator_matches_oracle(h, n, client, j):
    out = torch.full((n * n,), float("nan"), dtype=torch.float64, device="cuda")
    serve.fill_factor(77, client, j, n, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(n, n).T             # column-major storage
    ref = philox.factor(77, client, j, n, serving.scale(n))
    assert np.array_equal(got.view(np.int64), ref.view(np.int64))


SIZES = [32, 64, 33, 128, 32, 7]


def _schedule():
    a, c, l = serve.requests(9, len(SIZES), 4000.0, 0.01)
    return a, c, np.minimum(l, 6)       # short chains keep the CPU replay quick


def test_final_states_match_replay_and_timing(h):
    a, c, l = _schedule()
    srv = serve.Server(h, SIZES, seed=123)
    try:
        st, fi, ticks = srv.run(a, c, l)
        assert np.all(st >= a) and np.all(fi > st)
        assert ticks >= l.max() and ticks <= l.sum()
        prods = serving.products_per_client(len(SIZES), c, l)
        for cl, n in enumerate(SIZES):
            S, p = srv.state(cl)
            assert p == prods[cl]
            ref = serving.final_state(123, cl, n, int(p))
            err = np.linalg.norm(S - ref) / np.linalg.norm(ref)
            assert err <= 1e-13 * max(1, int(p)), (cl, n, p, err)
    finally:
        srv.close()


def test_results_identical_alone_and_in_the_mix(h):
    a, c, l = _schedule()
    srv = serve.Server(h, SIZES, seed=5)
    try:
        srv.run(a, c, l)
        mixed = {cl: srv.state(cl)[0] for cl in range(len(SIZES))}
        for cl in (0, 3):
            srv.reset()
            sel = c == cl
            srv.run(a[sel], c[sel], l[sel])
            alone, _ = srv.state(cl)
            assert np.array_equal(alone.view(np.int64), mixed[cl].view(np.int64)), cl
        # reset really restores the identity
        srv.reset()
        S, p = srv.state(2)
        assert p == 0 and np.array_equal(S, np.eye(SIZES[2]))
    finally:
        srv.close()


def test_budget_and_argument_errors(h):
    need = serve.bytes_needed(SIZES)
    factor = [(n * n * 8 + 255) // 256 * 256 for n in SIZES]
    resident = need - sum(factor)
    # the resident states plus the largest factor is the least budget
    with pytest.raises(bgemm.BgemmError) as e:
        serve.Server(h, SIZES, seed=1, budget=resident + max(factor) - 1)
    assert e.value.status == 4
    serve.Server(h, SIZES, seed=1, budget=resident + max(factor)).close()
    with pytest.raises(bgemm.BgemmError) as e:
        serve.Server(h, [32, 0], seed=1)
    assert e.value.status == 1
    srv = serve.Server(h, SIZES, seed=1, budget=need)
    try:
        with pytest.raises(bgemm.BgemmError) as e:
            srv.run([0.0, 0.0], [0, 9], [1, 1])
        assert e.value.status == 1
        st, fi, ticks = srv.run([], [], [])
        assert ticks == 0
    finally:
        srv.close()


@pytest.mark.parametrize("chain", [2, 3])
def test_graph_sweeps_equal_eager_sweeps(h, chain):
    """Lock-step sweeps replayed from a captured graph give the same bits as
    the same launches issued one by one, for 1, 2 and 3 replays (each count
    checked, with unrelated eager work and synchronisation in between), and
    match the CPU replay."""
    srv = serve.Server(h, SIZES, seed=17)
    A = torch.rand(4, 40, 40, dtype=torch.float64, device="cuda")
    Cx = torch.zeros_like(A)
    try:
        for sweeps in (1, 2, 3):
            srv.reset()
            t_eager = srv.sweeps(sweeps, chain, graph=False)
            eager = {cl: srv.state(cl) for cl in range(len(SIZES))}
            h.batched(A, A, Cx, 40, 40, 40, 1.0, 0.0)        # unrelated eager work
            torch.cuda.synchronize()
            srv.reset()
            t_graph = srv.sweeps(sweeps, chain, graph=True)
            h.batched(A, A, Cx, 40, 40, 40, 1.0, 0.0)
            torch.cuda.synchronize()
            assert t_eager > 0 and t_graph > 0
            for cl, n in enumerate(SIZES):
                S, p = srv.state(cl)
                E, pe = eager[cl]
                assert p == pe == sweeps * chain
                assert np.array_equal(S.view(np.int64), E.view(np.int64)), (sweeps, chain, cl)
        for cl, n in enumerate(SIZES[:3]):
            ref = serving.final_state(17, cl, n, 3 * chain)
            S, _ = srv.state(cl)
            assert np.linalg.norm(S - ref) <= 1e-13 * 3 * chain * np.linalg.norm(ref)
    finally:
        srv.close()


def test_sweeps_then_requests_continue_the_same_chain(h):
    # sweeps and requests share the product counter: 2 sweeps of 2, then a
    # request of 3 for client 1, equal the replay of 7 products
    srv = serve.Server(h, SIZES, seed=23)
    try:
        srv.sweeps(2, 2, graph=True)
        srv.run([0.0], [1], [3])
        S, p = srv.state(1)
        assert p == 7
        ref = serving.final_state(23, 1, SIZES[1], 7)
        assert np.linalg.norm(S - ref) <= 1e-12 * np.linalg.norm(ref)
    finally:
        srv.close()


def test_sweeps_argument_errors_and_zero_sweeps(h):
    srv = serve.Server(h, SIZES, seed=31)
    try:
        for sw, ch in ((-1, 2), (1, 0)):
            with pytest.raises(bgemm.BgemmError) as e:
                srv.sweeps(sw, ch, graph=False)
            assert e.value.status == 1
        for graph in (False, True):
            srv.sweeps(0, 3, graph=graph)            # nothing replayed
            for cl, n in enumerate(SIZES):
                S, p = srv.state(cl)
                assert p == 0 and np.array_equal(S, np.eye(n))
    finally:
        srv.close()


def test_lockstep_and_tight_memory_give_the_same_states(h):
    """The lock-step policy and a budget that admits one large factor at a
    time change only when products run, not what they compute: final states
    are bit-identical to continuous batching with no memory limit."""
    a, c, l = _schedule()
    ref = serve.Server(h, SIZES, seed=31)
    try:
        ref.run(a, c, l)
        want = {cl: ref.state(cl) for cl in range(len(SIZES))}
        _, _, waits = ref.memory_stats()
        assert waits == 0
    finally:
        ref.close()
    need = serve.bytes_needed(SIZES)
    factor = [(n * n * 8 + 255) // 256 * 256 for n in SIZES]
    tight = need - sum(factor) + max(factor) + factor[0]
    for policy, budget in ((serve.POLICY_LOCKSTEP, 0), (serve.POLICY_CONTINUOUS, tight),
                           (serve.POLICY_LOCKSTEP, tight)):
        srv = serve.Server(h, SIZES, seed=31, budget=budget)
        try:
            srv.set_policy(policy)
            st, fi, ticks = srv.run(a, c, l)
            assert np.all(st >= a) and np.all(fi > st)
            pool, peak, waits = srv.memory_stats()
            assert peak <= pool
            if budget:
                assert pool == max(factor) + factor[0] and waits > 0
            for cl in range(len(SIZES)):
                S, p = srv.state(cl)
                W, pw = want[cl]
                assert p == pw and np.array_equal(S.view(np.int64), W.view(np.int64)), (policy, cl)
        finally:
            srv.close()


def test_one_variable_size_launch_per_tick_gives_the_same_states(h):
    """Ticks issued as one bg_dgemm_vbatched over every product (instead of
    one bg_dgemm_batched per client size) compute the same products: final
    states are bit-identical, under both policies."""
    a, c, l = _schedule()
    ref = serve.Server(h, SIZES, seed=41)
    try:
        ref.run(a, c, l)
        want = {cl: ref.state(cl) for cl in range(len(SIZES))}
    finally:
        ref.close()
    for policy in (serve.POLICY_CONTINUOUS, serve.POLICY_LOCKSTEP):
        srv = serve.Server(h, SIZES, seed=41)
        try:
            with pytest.raises(bgemm.BgemmError):
                srv.set_tick_launch(2)
            srv.set_tick_launch(serve.TICK_VBATCHED)
            srv.set_policy(policy)
            st, fi, ticks = srv.run(a, c, l)
            assert np.all(st >= a) and np.all(fi > st)
            for cl in range(len(SIZES)):
                S, p = srv.state(cl)
                W, pw = want[cl]
                assert p == pw and np.array_equal(S.view(np.int64), W.view(np.int64)), (policy, cl)
        finally:
            srv.close()


@pytest.mark.parametrize("extra", [[200, 130], [200, 130] + [65] * 70])
def test_sizes_sharing_a_launch_give_the_same_states(h, extra):
    """Nineteen or twenty short size groups (more than one launch holds), on
    the narrow tiles and, with the 65s, on the wide ones, next to a group that
    fills the chip by itself (520 clients of 40): the same bits as one
    variable-size launch per tick, in requests and in captured sweeps."""
    sizes = list(range(1, 18)) + extra + [40] * 520
    nc = len(sizes)
    got = []
    for mode in (serve.TICK_PER_SIZE, serve.TICK_VBATCHED):
        srv = serve.Server(h, sizes, seed=43)
        try:
            srv.set_tick_launch(mode)
            srv.run(np.zeros(nc), np.arange(nc), np.full(nc, 3))
            got.append([srv.state(c)[0] for c in range(nc)])
        finally:
            srv.close()
    srv = serve.Server(h, sizes, seed=43)
    try:
        srv.sweeps(3, 1, True)
        got.append([srv.state(c)[0] for c in range(nc)])
    finally:
        srv.close()
    for c in range(nc):
        for other in got[1:]:
            assert np.array_equal(got[0][c].view(np.int64), other[c].view(np.int64)), sizes[c]
    ref = serving.final_state(43, 18, 130, 3)
    assert np.linalg.norm(got[0][18] - ref) <= 3e-13 * np.linalg.norm(ref)
