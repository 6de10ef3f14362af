"""GPU parity of the TIES trim over block lengths, expert counts and
densities: the catalog's thresholds and sums of squares, and both TIES merges,
against the CPU oracle, bit for bit."""

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _run_all, _say, mp  # noqa: F401  (mp: the module fixture)
from workloads import FamilySpec

pytestmark = pytest.mark.gpu


def _spread_family(be, dtype, K, seed):
    """Tensors that end inside, at and one chunk past a block, and deltas that
    put the k-th largest everywhere: normal; log-uniform over 24 binades (far
    below the block maximum at high densities); nine tenths zero; a few huge
    outliers; and, in fp32, magnitudes that share their top 16 bits (more of
    them than a histogram row lists)."""
    v = 4 if dtype == "f32" else 8
    t = tuple((f"t{j}", (n,)) for j, n in enumerate((3 * be + v, be, be - v if be > v else v, v, 2 * be)))
    spec = FamilySpec("spread", t, dtype, be, K, ())
    P = sum(n for _, (n,) in t)
    rng = np.random.default_rng(seed)
    sign = lambda: rng.choice([-1.0, 1.0], P)  # noqa: E731
    kinds = [rng.normal(0.0, 1e-3, P),
             np.exp2(rng.uniform(-30.0, -6.0, P)) * sign(),
             np.where(rng.random(P) < 0.1, rng.normal(0.0, 1e-3, P), 0.0),
             np.where(rng.random(P) < 0.01, rng.normal(0.0, 1.0, P), rng.normal(0.0, 1e-4, P)),
             1e-3 * (1.0 + rng.integers(0, 1 << 14, P) * 2.0 ** -23) * sign()]
    deltas = [kinds[(i + seed) % len(kinds)].astype(np.float32) for i in range(K)]
    if dtype == "f32":  # a zero base keeps the fp32 patterns
        return spec, np.zeros(P, np.float32), deltas
    base = oracle.round_bf16(rng.normal(0.0, 0.02, P).astype(np.float32))
    x0 = (base.astype(np.uint32) << 16).view(np.float32)
    return spec, base, [oracle.round_bf16(x0 + d) for d in deltas]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("be,K", [(64, 3), (512, 5), (520, 2), (1024, 7), (1032, 1), (2048, 9), (2056, 4),
                                  (2048, 1), (4096, 1), (4096, 6), (4096, 17)])
def test_trim_over_block_lengths(mp, dtype, be, K):  # noqa: F811
    spec, base, exps = _spread_family(be, dtype, K, seed=be + K)
    for density in (0.05, 0.2, 0.5, 0.95, 1.0):
        _say(f"case {dtype} block {be} K {K} density {density}")
        _run_all(mp, spec, base, exps, "ties_tau", [0.5, 1.0], density=density, lam=1.0)
        _run_all(mp, spec, base, exps, "ties", [0.3, 1.0], density=density, lam=0.7)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_trim_explicit_deltas(mp, dtype):  # noqa: F811
    for be, K in ((512, 3), (1024, 4), (2048, 2), (4096, 5)):
        spec, base, exps = _spread_family(be, "f32", K, seed=be)
        if dtype == "bf16":
            spec = FamilySpec("spread", tuple((n, (max(8, s // 8 * 8),)) for n, (s,) in spec.tensors), "bf16", be, K, ())
            P = sum(s for _, (s,) in spec.tensors)
            base = oracle.round_bf16(np.resize(base, P))
            exps = [oracle.round_bf16(np.resize(x, P)) for x in exps]
        _say(f"case deltas {dtype} block {be} K {K}")
        _run_all(mp, spec, base, exps, "ties_tau", [0.5], delta=True, density=0.3, lam=1.0)
        _run_all(mp, spec, base, exps, "ties", [0.5], delta=True, density=0.3, lam=1.0)


@pytest.mark.parametrize("be,K", [(512, 3), (1024, 6), (4096, 9)])
def test_in_merge_trim_from_pinned_experts(mp, be, K):  # noqa: F811
    """Pinned experts keep the form that reads every byte once, also where
    device experts take the one that reads a block twice."""
    spec, base, exps = _spread_family(be, "bf16", K, seed=7 * be + K)
    _say(f"case pinned block {be} K {K}")
    _run_all(mp, spec, base, exps, "ties", [0.4, 1.0], residency=mp.MP_HOST_PINNED, density=0.2, lam=1.0)
