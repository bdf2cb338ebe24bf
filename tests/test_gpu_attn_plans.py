"""GPU tests of the attention's split plans at the sizes where they change:
key-block and ring edges, the unsplit limit, the last split's share, one and
several query groups, a batch in one and in two rounds of the chip.

The reference is the same attention in float64.  Tolerance: probabilities and
partial outputs are rounded to bf16 (2^-9 each) around values of order one, so
an output is off by less than 2^-8 of the largest value it mixes, about 4.
"""
import math
import random

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2606_27550_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

D = 128
THETA = 10000.0
SCALE = 1 / math.sqrt(D)
TOL = 4 * 2.0 ** -8


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27550_amd import api as _api
    return _api


def tree(T):
    return synth.uniform_attach_tree(31, T, min(T - 1, 5)) if T > 1 else [-1]


def normal(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def rope(x, pos):
    c = torch.arange(D // 2, device="cuda", dtype=torch.float64)
    a = pos.double()[:, None] * THETA ** (-2 * c / D)
    lo, hi = x[..., :64], x[..., 64:]
    cos, sin = a.cos()[:, None], a.sin()[:, None]
    return torch.cat((lo * cos - hi * sin, hi * cos + lo * sin), -1)


def reference(parent, q, k, v, kc, vc, L):
    """out in float64; appends to kc / vc."""
    T, Hq, Hkv = q.shape[0], q.shape[1], k.shape[1]
    depth, seen = [0] * T, torch.eye(T, dtype=torch.bool)
    for i in range(1, T):
        depth[i] = depth[parent[i]] + 1
        seen[i] |= seen[parent[i]]
    pos = L + torch.tensor(depth, device="cuda")
    kc[:, L:L + T] = rope(k.double(), pos).to(torch.bfloat16).transpose(0, 1)
    vc[:, L:L + T] = v.transpose(0, 1)
    qr = rope(q.double(), pos)
    out = torch.empty((T, Hq, D), dtype=torch.float64, device="cuda")
    for h in range(Hq):
        g = h // (Hq // Hkv)
        z = qr[:, h].contiguous() @ kc[g, :L + T].double().t().contiguous() * SCALE
        z[:, L:] = z[:, L:].masked_fill(~seen.cuda(), -math.inf)
        out[:, h] = torch.softmax(z, 1) @ vc[g, :L + T].double()
    return out


@pytest.mark.parametrize("T,L,Hq,Hkv", [
    (1, 0, 2, 2), (1, 31, 2, 2), (7, 32, 4, 2), (32, 96, 2, 2), (33, 127, 2, 2),
    (27, 128, 2, 2), (27, 160, 2, 2),      # ring rounds: 4 and 5 prefix blocks
    (31, 321, 2, 2), (32, 321, 2, 2),      # 11 and 12 blocks: the unsplit limit
    (31, 609, 2, 2), (32, 609, 2, 2),      # 20 and 21 blocks
    (1, 1023, 3, 3), (1, 1024, 3, 1), (128, 1500, 2, 1), (129, 900, 1, 1), (256, 700, 2, 1),
    (64, 5000, 5, 5), (5, 8191, 28, 4),
])
def test_lone_sequence(api, T, L, Hq, Hkv):
    print("[gpu-test] attention plan", T, L, Hq, Hkv, flush=True)
    parent = tree(T)
    bank = api.Bank([parent])
    q, k, v = normal(1, T, Hq, D), normal(2, T, Hkv, D), normal(3, T, Hkv, D)
    kc, vc = normal(4, Hkv, L + T + 3, D), normal(5, Hkv, L + T + 3, D)
    rk, rv = kc.clone(), vc.clone()
    out = torch.full_like(q, float("nan"))
    ws = torch.empty(max(api.tree_attn_workspace(T, Hq, Hkv, D, L), 256), dtype=torch.uint8, device="cuda")
    api.tree_attn(bank, 0, q, k, v, kc, vc, L, SCALE, THETA, out, ws)
    ref = reference(parent, q, k, v, rk, rv, L)
    assert float((out.double() - ref).abs().max()) <= TOL
    assert torch.equal(vc, rv)
    # the library's angles and torch's differ in the last bits of fp64: keys
    # agree but for ties of the bf16 rounding
    assert float((kc.double() - rk.double()).abs().max()) <= 2.0 ** -6
    assert float((kc != rk).float().mean()) < 1e-4


@pytest.mark.parametrize("B,Hq,Hkv,lo,hi", [
    (2, 4, 4, 0, 700), (3, 8, 2, 600, 5000), (16, 8, 2, 10, 4000),
    (16, 32, 32, 5, 1500),     # streams fill the chip: two rounds allowed
    (5, 28, 4, 2000, 2100),
])
def test_batch_host_and_device_plans(api, B, Hq, Hkv, lo, hi):
    """Both batched forms against the reference, and equal to each other."""
    print("[gpu-test] batch plan", B, Hq, Hkv, lo, hi, flush=True)
    trees = [tree(n) for n in (1, 8, 27, 64, 128)]
    r = random.Random(B * hi)
    topo = [r.randrange(5) for _ in range(B)]
    lens = [r.randint(lo, hi) for _ in range(B)]
    cap = max(lens) + 128
    off = np.concatenate([[0], np.cumsum([len(trees[t]) for t in topo])]).tolist()
    q, k, v = normal(1, off[-1], Hq, D), normal(2, off[-1], Hkv, D), normal(3, off[-1], Hkv, D)
    kcs = [normal(10 + b, Hkv, cap, D) for b in range(B)]
    vcs = [normal(40 + b, Hkv, cap, D) for b in range(B)]
    bank = api.Bank(trees)
    res = []
    for device in (False, True):
        kc, vc = [x.clone() for x in kcs], [x.clone() for x in vcs]
        out = torch.full_like(q, float("nan"))
        if device:
            n = api.tree_attn_batched_device_workspace(bank, B, Hq, Hkv, D, cap)
            ws = torch.empty(n, dtype=torch.uint8, device="cuda")
            dev = [torch.tensor(x, dtype=torch.int32, device="cuda") for x in (topo, lens, off)]
            api.tree_attn_batched_device(bank, *dev, q, k, v, kc, vc, SCALE, THETA, out, ws)
        else:
            n = api.tree_attn_batched_workspace(B, 128, Hq, Hkv, D, max(lens))
            ws = torch.empty(n, dtype=torch.uint8, device="cuda")
            api.tree_attn_batched(bank, topo, lens, q, k, v, kc, vc, SCALE, THETA, out, ws)
        res.append((out, kc, vc))
    assert torch.equal(res[0][0], res[1][0])
    for b in range(B):
        s, e = off[b], off[b + 1]
        ref = reference(trees[topo[b]], q[s:e], k[s:e], v[s:e], kcs[b], vcs[b], lens[b])
        assert float((res[0][0][s:e].double() - ref).abs().max()) <= TOL
        assert torch.equal(res[0][1][b], res[1][1][b]) and torch.equal(res[0][2][b], res[1][2][b])
        assert torch.equal(res[0][2][b], vcs[b])
        assert float((res[0][1][b].double() - kcs[b].double()).abs().max()) <= 2.0 ** -6


@pytest.mark.parametrize("T,G,Hkv,L,step", [
    (128, 32, 8, 40, 0),      # unsplit: more attend workgroups than disjoint rows could take
    (128, 1, 8, 3000, 64),    # split: more merge blocks
])
def test_device_batch_sequences_that_share_rows(api, T, G, Hkv, L, step):
    """Device-planned sequences whose row ranges overlap (a sequence without
    work between two of them has a range that ends below its start): every
    sequence is computed, whatever the grids were sized for.  All have the same
    queries, keys and caches; where rows of different nodes coincide, only those
    that one sequence alone writes are compared."""
    print("[gpu-test] device batch of sequences that share rows", T, G, Hkv, flush=True)
    n = 8
    parent = [-1] + [0] * (T - 1)
    bank = api.Bank([parent])
    rows = T + step * (n - 1)
    q, k, v = normal(1, T, G * Hkv, D), normal(2, T, Hkv, D), normal(3, T, Hkv, D)
    if step:   # equal rows, so that every sequence's tree has the same
        q, k, v = (x[:1].repeat(rows, 1, 1) for x in (q, k, v))
    kc0, vc0 = normal(4, Hkv, L + T, D), normal(5, Hkv, L + T, D)
    kc, vc = [kc0.clone() for _ in range(2 * n)], [vc0.clone() for _ in range(2 * n)]
    out = torch.full_like(q, float("nan"))
    off = [x for b in range(n) for x in (step * b, step * b + T)] + [0]
    dev = [torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([0, -1] * n, [L] * 2 * n, off)]
    ws = torch.empty(api.tree_attn_batched_device_workspace(bank, 2 * n, G * Hkv, Hkv, D, L + T),
                     dtype=torch.uint8, device="cuda")
    api.tree_attn_batched_device(bank, *dev, q, k, v, kc, vc, SCALE, THETA, out, ws)
    rk, rv = kc0.clone(), vc0.clone()
    ref = reference(parent, q[:T], k[:T], v[:T], rk, rv, L)
    for b in range(2 * n):
        assert torch.equal(vc[b], vc0 if b % 2 else rv), b
        assert torch.equal(kc[b], kc0 if b % 2 else kc[0]), b
    if step == 0:
        assert float((out.double() - ref).abs().max()) <= TOL
    else:   # the rows that one sequence alone writes
        assert float((out[:step].double() - ref[:step]).abs().max()) <= TOL
        assert float((out[-step:].double() - ref[-step:]).abs().max()) <= TOL
