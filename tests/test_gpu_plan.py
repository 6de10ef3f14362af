"""Algorithm 1 on the device against the oracle's literal sort + greedy, where
the plan's routes change: unit counts around the one-workgroup plan's limit and
the marking pass's uid range, candidate lists around and past what stays in
registers, ties of every kind, zeros, and the tensor-level plan past both."""

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _say, mp  # noqa: F401  (mp: the module fixture)

pytestmark = pytest.mark.gpu


def _scores(kind, n, rng):
    if kind == "spread":
        S = rng.lognormal(-14.0, 2.0, n)
        S[rng.random(n) < 0.2] = 0.0
    elif kind == "equal":
        S = np.full(n, 2.5e-3)
    elif kind == "few":
        S = rng.choice([0.0, 1e-4, 2.5e-3, 7e-2, 1.0], n)
    elif kind == "near":  # share all but the low bits of the score
        return (np.float32(1.0).view(np.uint32) + rng.integers(0, 3000, n).astype(np.uint32)).view(np.float32)
    else:  # "wide": every exponent, subnormal squares and infinity among them
        S = np.where(rng.random(n) < 0.001, np.inf, np.exp2(rng.uniform(-140.0, 120.0, n)))
    return S.astype(np.float32)


def _plans(mp, numel, be, K, S, budgets, flags_list=(0, 1, 2, 3), w=None):  # noqa: F811
    import torch
    L = mp.Layout(numel, be, mp.MP_BF16)
    blocks = oracle.Blocks(numel, be)
    mask = torch.empty(blocks.G, dtype=torch.int32, device="cuda")
    dev = None if S is None else torch.from_numpy(S).cuda()
    w = w or [1.0] * K
    for flags in flags_list:
        for B in budgets:
            st = mp.mp_plan(L, K, dev, w, B, mask, flags=flags)
            m_orc, o = oracle.plan(blocks, "bf16", K, S, w, B, flags=flags)
            assert np.array_equal(mask.cpu().numpy().view(np.uint32), m_orc), f"B={B} flags={flags}"
            assert (st["cost_bytes"], st["n_selected"], st["digest"], st["full_bytes"], st["n_units"]) == \
                (o["cost"], o["n_selected"], o["digest"], o["full_bytes"], blocks.G * K)


def _budgets(full, rng):
    return sorted({0, 16, full // 1000, full // 4, full // 2, full - full // 50, full - 1, full, full + 5}
                  | {int(x) for x in rng.integers(0, full, 3)})


# (full blocks, short tensors, K): 1024/1025 and 8191/8192/8193 units; 4096-uid ranges on both
# sides; 300 thousand units; 8,192 and more listed candidates
@pytest.mark.parametrize("blocks,short,K", [(1020, 4, 1), (1021, 4, 1), (8191, 0, 1), (4092, 4, 2), (8190, 3, 1), (8000, 193, 1), (2000, 60, 5),
                                            (9000, 300, 32), (70_000, 500, 4), (3000, 2048, 4), (3000, 2049, 4)])
def test_plan_routes(mp, blocks, short, K):  # noqa: F811
    be = 64
    rng = np.random.default_rng(blocks + short)
    numel = [be * blocks] + [int(x) * 8 for x in rng.integers(1, be // 8, short)]
    full = 2 * K * sum(numel)
    n = (blocks + short) * K
    for kind in ("spread", "equal", "few", "near", "wide"):
        _say(f"case {blocks} blocks, {short} short, K {K}, {kind} scores")
        few = kind != "spread" and n > 50_000
        _plans(mp, numel, be, K, _scores(kind, n, rng), _budgets(full, rng), (0, 3) if few else (0, 1, 2, 3),
               None if kind != "few" else [0.5 + 0.25 * (i % 3) for i in range(K)])


@pytest.mark.parametrize("T,K", [(2730, 3), (2731, 3), (300, 32)])
def test_tensor_level_plan_routes(mp, T, K):  # noqa: F811
    rng = np.random.default_rng(T)
    numel = [int(x) * 8 for x in rng.integers(0, 300, T)]
    full = 2 * K * sum(numel)
    _say(f"case {T} tensors, K {K}")
    _plans(mp, numel, 64, K, None, _budgets(full, rng), w=[1.0 + (i % 3) for i in range(K)])


@pytest.mark.parametrize("blocks", [376_989, 250])
def test_plan_runs_beside_a_merge(mp, blocks):  # noqa: F811
    """A plan (of 1.5M units, of 1,000) on a second stream ends while a merge of 18 GB (3 ms) still runs on
    the first: its workgroups fit into the slots that the merge's waves leave one
    by one.  Its mask is the one of a plan alone."""
    import torch
    be, K, G = 4096, 4, 376_989
    L = mp.Layout([be * G], be, mp.MP_BF16)
    base, *exps = [torch.zeros(be * G, dtype=torch.bfloat16, device="cuda") for _ in range(1 + K)]
    out = torch.empty_like(base)
    P = mp.Layout([be * blocks], be, mp.MP_BF16)  # what is planned
    S = torch.from_numpy(_scores("spread", blocks * K, np.random.default_rng(2))).cuda()
    alone, beside = (torch.empty(blocks, dtype=torch.int32, device="cuda") for _ in range(2))
    every = torch.full((G,), (1 << K) - 1, dtype=torch.int32, device="cuda")
    tau = torch.ones(G * K, dtype=torch.int32, device="cuda")
    budget = be * blocks * K
    side = torch.cuda.Stream()
    st = mp.mp_plan(P, K, S, [1.0] * K, budget, alone)
    mp.mp_merge_ties_tau(L, base, exps, every, tau, 1.0, out)
    torch.cuda.synchronize()
    early = 0
    for _ in range(5):
        done = torch.cuda.Event()
        mp.mp_merge_ties_tau(L, base, exps, every, tau, 1.0, out)
        done.record()
        assert mp.mp_plan(P, K, S, [1.0] * K, budget, beside, stream=side) == st  # returns when its stream has ended
        early += not done.query()
        torch.cuda.synchronize()
        assert torch.equal(beside, alone)
    assert early >= 3, f"the plan ended before the merge in {early} of 5 tries"
