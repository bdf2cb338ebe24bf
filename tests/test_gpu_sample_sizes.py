"""GPU tests of the sampling path's kernels at the vocabulary sizes where their
forms change: a thread's share of one entry, chunk lengths odd and even, the
largest row kept in LDS at each number of entries a thread and the first beyond
it, one and two slabs of a row in either width of load and both lengths of slab.
Decisions against the oracle (inputs redrawn until they are clear), statistics
at the bounds of tests/test_gpu_kernels.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import entmtp_oracle as orc  # noqa: E402
from paper_2606_27550_amd import synth  # noqa: E402
from tests import test_gpu_kernels as kern  # noqa: E402
from tests import test_gpu_speculative as spec  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27550_amd import api as _api
    return _api


@pytest.mark.parametrize("V", [2, 1023, 1025, 2048, 2049, 8192, 8193, 30723, 32768, 32769, 50001])
def test_stochastic_vocabulary_sizes(api, V):
    g = np.random.default_rng(V)
    parent = synth.uniform_attach_tree(17, 24, 3)
    for rep in range(3):
        z, q, tok, ua, us, ref = spec.make_inputs(g, parent, V, 1 / 0.7)
        print("[gpu-test] stochastic V", V, "rep", rep, "tests", len(ref[4]) - 1, flush=True)
        a, path, bonus = spec.run(api, parent, z, q, tok, ua, us, 1 / 0.7)
        assert (a, bonus) == (ref[0], ref[2])
        assert path[: a + 1] == list(ref[1])


@pytest.mark.parametrize("V", [1, 3, 4, 2047, 2048, 2052, 4095, 4097, 8192, 8196, 16384, 16385, 32768, 32772,
                               65537])
def test_logit_stats_slabs(api, V):
    print("[gpu-test] logit_stats V", V, flush=True)
    g = np.random.default_rng(V)
    z = g.normal(0, 2.5, (3, V)).astype(np.float32)
    z[1, : V // 2] = -np.inf   # masked entries
    z[2, V - 1] = 40.0         # the last entry wins
    kern.check_stats(kern.run_stats(api, z, 1.0), orc.logit_stats(z))


@pytest.mark.parametrize("V", [3, 1000, 1500, 31999])
def test_stochastic_rows_end_at_the_vocabulary(api, V):
    """What lies behind the last row of the logits and of the draft
    probabilities has no part in a residual: with large negative values there,
    the sibling tested after a rejection passes as in the oracle.  (Child 1
    carries the token the draft overrates most, child 2 the one it underrates
    most.)"""
    g = np.random.default_rng(V)
    parent = [-1, 0, 0, 2]
    T, pad = len(parent), 40000
    bank = api.Bank([parent])
    checked = 0
    for rep in range(8):
        z, q, tok, _, us, _ = spec.make_inputs(g, parent, V, 1.0)
        p = spec.softmax(z[0].astype(np.float64))
        tok[1], tok[2] = np.argmax(q[0] / p), np.argmax(p - q[0])
        ua = np.array([0.5, 0.999, 0.01, 0.5], np.float32)
        ref = orc.accept_stochastic(parent, tok, *(x.astype(np.float64) for x in (z, q)), 1.0,
                                    *(x.astype(np.float64) for x in (ua, us)))
        _, target, lo, hi = ref[4][-1]
        clear = (min(target - lo, hi - target) > spec.DRAW_MARGIN
                 and all(abs(e[1] - e[2]) > spec.MARGIN_REL * max(e[1], e[2]) + spec.MARGIN_ABS
                         for e in ref[4][:-1]))
        if not clear or list(ref[1][:2]) != [0, 2]:
            continue
        print("[gpu-test] stochastic row ends V", V, "rep", rep, flush=True)
        checked += 1

        def wide(a, rest):
            t = torch.full((T * V + pad,), rest, device="cuda")
            t[: T * V] = torch.from_numpy(a.reshape(-1)).cuda()
            return t[: T * V].view(T, V)

        zd, qd = wide(z, 50.0), wide(q, -1e4)
        H, p1 = torch.empty(T, device="cuda"), torch.empty(T, device="cuda")
        am, path = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (T, bank.D[0] + 1))
        a, bonus = (torch.full((1,), -3, dtype=torch.int32, device="cuda") for _ in range(2))
        api.logit_stats(zd, 1.0, H, p1, am)
        f = lambda x: torch.from_numpy(x).cuda()   # noqa: E731
        api.accept_stochastic(bank, 0, spec.dev_i32(tok), zd, qd, 1.0, am, p1, f(ua), f(us),
                              torch.empty(V, device="cuda"), a, path, bonus)
        assert (int(a), int(bonus)) == (ref[0], ref[2])
        assert path.tolist()[: ref[0] + 1] == list(ref[1])
    assert checked >= 3


@pytest.mark.parametrize("V", [32000, 50001])
def test_logit_stats_of_large_logits(api, V):
    """A lone large logit has probability one at any temperature: its own term
    is exactly one (temperature times the logit alone would bring a rounding of
    its own size, 1.5e-5 at 200), the others sum to less than 1e-8."""
    print("[gpu-test] logit_stats of large logits V", V, flush=True)
    g = np.random.default_rng(V)
    z = g.normal(0, 2.5, (40, V)).astype(np.float32)
    top = g.integers(0, V, 40)
    z[np.arange(40), top] = g.uniform(100, 300, 40).astype(np.float32)
    for it in (1 / 0.7, 0.9):
        H, p1, am = kern.run_stats(api, z, it)
        np.testing.assert_array_equal(am, top)
        assert (np.abs(p1 - 1) <= 1e-7).all() and (np.abs(H) <= 1e-6).all()
