"""Tensor-scope TIES thresholds on the device against the CPU oracle, bit for
bit, where the one-pass route can go wrong: tensor sizes around its list-all
limit and its slices, repeated values, samples that mislead, lists that
overflow, blocks too long for it, and a workspace without room for its lists."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import to_dev
from tests.test_gpu_parity import _say, mp  # noqa: F401  (mp: the module fixture)

pytestmark = pytest.mark.gpu


def _check(mp, dtype, be, numel, base, exps, mask, density, delta=False):  # noqa: F811
    import torch
    L = mp.Layout(numel, be, mp.MP_F32 if dtype == "f32" else mp.MP_BF16)
    blocks = oracle.Blocks(numel, be)
    K = len(exps)
    tau = torch.full((blocks.G * K,), -1, dtype=torch.int32, device="cuda")
    m = torch.from_numpy(mask.view(np.int32)).to("cuda")
    mp.mp_ties_tensor_thresholds(L, to_dev(base, dtype), [to_dev(e, dtype) for e in exps], m, density, tau, delta=delta)
    want = oracle.expand_tensor_thresholds(
        blocks, oracle.ties_tensor_thresholds(blocks, dtype, base, exps, mask, density, delta=delta))
    assert np.array_equal(tau.cpu().numpy().view(np.uint32), want), f"{dtype} be={be} density={density}"


def _sampled(dtype, numel, be):
    """The elements that the sample reads of whole-mask units: of block g (over
    all tensors) slice g mod 32 of max(1, 1/32 of a full block) 16-byte chunks,
    the first slice where the block is too short to have that one."""
    v = 4 if dtype == "f32" else 8
    segc, seen, g = max(1, be // v // 32), [], 0
    for n in numel:
        for x in range(0, n, be):
            nch = min(be, n - x) // v
            first = g % 32 * segc
            first = 0 if nch <= first else first
            c = np.arange(nch)
            seen.append(np.repeat((c >= first) & (c < first + segc), v))
            g += 1
    return np.concatenate(seen)


def _encode(dtype, deltas, seed):
    deltas = [d.astype(np.float32) for d in deltas]
    P = len(deltas[0])
    if dtype == "f32":  # a zero base keeps the fp32 patterns
        return np.zeros(P, np.float32), deltas
    base = oracle.round_bf16(np.random.default_rng(seed).normal(0.0, 0.02, P).astype(np.float32))
    x0 = (base.astype(np.uint32) << 16).view(np.float32)
    return base, [oracle.round_bf16(x0 + d) for d in deltas]


def _misleading(dtype, numel, be, seed):
    """Large only where the sample reads (it sees nothing else), and large only
    where it does not."""
    rng = np.random.default_rng(seed)
    seen = _sampled(dtype, numel, be)
    return [np.where(where, 1.0, 1e-3) * rng.normal(0.0, 1.0, len(seen)) for where in (seen, ~seen)]


def _family(dtype, numel, be, seed):
    """Seven experts: normal, a few repeated values, mostly zero, all equal, the
    two that mislead the sample, and magnitudes that share their top 16 bits."""
    P = sum(numel)
    rng = np.random.default_rng(seed)
    sign = rng.choice([-1.0, 1.0], P)
    deltas = [rng.normal(0.0, 1e-3, P), rng.choice([0.5, 1.0, 1.5], P) * 2.0 ** -10 * sign,
              np.where(rng.random(P) < 0.05, rng.normal(0.0, 1e-3, P), 0.0), np.full(P, 2.0 ** -9),
              *_misleading(dtype, numel, be, seed + 1),
              1e-3 * (1.0 + rng.integers(0, 1 << 14, P) * 2.0 ** -23) * sign]
    return _encode(dtype, deltas, seed + 2)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("be", [64, 520, 4096, 8192])
def test_tensor_thresholds_edges(mp, dtype, be):  # noqa: F811
    numel = [8, 3576, 3584, 3592, 8184, 8192, 8200, 17 * be + 8, 300_000, 16 * be, 40 * be - 8]
    base, exps = _family(dtype, numel, be, seed=be)
    K, G = len(exps), oracle.Blocks(numel, be).G
    rng = np.random.default_rng(be)
    some = rng.integers(0, 1 << K, G).astype(np.uint32)
    for mask in (some, np.full(G, (1 << K) - 1, np.uint32), np.zeros(G, np.uint32)):
        for density in (0.0, 1e-6, 0.01, 0.2, 0.5, 0.9, 1.0):
            _say(f"case {dtype} block {be} density {density}")
            _check(mp, dtype, be, numel, base, exps, mask, density)
            assert (mp.mp_ties_tensor_left() == -1) == (be > 4096)  # longer blocks have no one-pass route
    _check(mp, dtype, be, numel, base, exps, some, 0.2, delta=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("be", [64, 520, 4096])
def test_misleading_samples_are_left_over(mp, dtype, be):  # noqa: F811
    """Samples that see only the large deltas, or none of them: every pair's k-th
    largest lies outside its bracket (below it, above it), and the digit passes
    finish both pairs.  A normal expert beside them needs no such pass."""
    numel = [300_000]
    rng = np.random.default_rng(5)
    base, exps = _encode(dtype, [*_misleading(dtype, numel, be, 6), rng.normal(0.0, 1e-3, numel[0])], 7)
    G = oracle.Blocks(numel, be).G
    for density in (0.01, 0.2):
        for bits in (1, 2, 4, 7):
            _say(f"case {dtype} block {be} density {density} experts {bits:03b}")
            mask = np.full(G, bits, np.uint32)
            _check(mp, dtype, be, numel, base, exps, mask, density)
            assert mp.mp_ties_tensor_left() == bin(bits & 3).count("1")


def test_tensor_thresholds_without_lists(mp):  # noqa: F811
    """A workspace limit that leaves no room for the lists: the library gives them
    back, every pair takes the digit passes, and the thresholds are the same."""
    be, numel = 4096, [300_000, 8192]
    base, exps = _family("bf16", numel, be, seed=1)
    mask = np.full(oracle.Blocks(numel, be).G, 127, np.uint32)
    mp.mp_release()
    _check(mp, "bf16", be, numel, base, exps, mask, 0.2)
    assert mp.mp_ties_tensor_left() >= 0
    held = mp.mp_workspace_bytes()
    lists = 4 * len(exps) * (8192 + 32 * 547 + 300_000 // 256 + 8192)
    try:
        mp.mp_set_workspace_limit(held)
        _check(mp, "bf16", be, numel[::-1], base, exps, mask, 0.2)  # its table takes the lists' place
        assert mp.mp_ties_tensor_left() == -1
        assert mp.mp_workspace_bytes() < held and held - lists < mp.mp_workspace_bytes()
    finally:
        mp.mp_set_workspace_limit(0)
    _check(mp, "bf16", be, numel, base, exps, mask, 0.3)
    assert mp.mp_ties_tensor_left() >= 0


def _normal(dtype, P, K, seed):
    rng = np.random.default_rng(seed)
    base = rng.normal(0.0, 0.02, P).astype(np.float32)
    exps = [(base + rng.normal(0.0, 1e-3 * (1 + i), P)).astype(np.float32) for i in range(K)]
    return (base, exps) if dtype == "f32" else (oracle.round_bf16(base), [oracle.round_bf16(x) for x in exps])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("numel", [[16_384] * 3 + [98_304, 393_216], [1 << 20, 2_359_296], [4 << 20]])
def test_normal_deltas_leave_no_pair(mp, dtype, numel):  # noqa: F811
    """Normal base and deltas: every bracket holds its k-th largest and fits its
    list, at any density and share of blocks (fp32 patterns are nearly all
    listed, so this is what the lists' room is measured by)."""
    be, K = 4096, 2
    base, exps = _normal(dtype, sum(numel), K, seed=len(numel))
    G = oracle.Blocks(numel, be).G
    half = np.random.default_rng(3).integers(0, 1 << K, G).astype(np.uint32)
    for mask in (np.full(G, (1 << K) - 1, np.uint32), half):
        for density in (0.05, 0.2, 0.5, 0.8):
            _say(f"case {dtype} {numel} density {density}")
            _check(mp, dtype, be, numel, base, exps, mask, density)
            assert mp.mp_ties_tensor_left() == 0


def test_large_lists_are_given_back(mp):  # noqa: F811
    """Lists past what the library keeps between calls (1300 tensors of 16,384
    elements x 32 experts: 2.1 GB) are used and freed: what a call holds
    afterwards beyond the pairs' fixed scratch stays below 1 GiB."""
    import torch
    be, K, numel = 4096, 32, [16_384] * 1300
    base, exps = _normal("bf16", sum(numel), 1, seed=9)
    L, G = mp.Layout(numel, be, mp.MP_BF16), oracle.Blocks(numel, be).G
    b, e = to_dev(base, "bf16"), to_dev(exps[0], "bf16")
    mask = torch.full((G,), -1, dtype=torch.int32, device="cuda")
    one = torch.empty(G, dtype=torch.int32, device="cuda")
    mp.mp_release()
    mp.mp_ties_tensor_thresholds(L, b, [e], mask, 0.2, one)
    before = mp.mp_workspace_bytes()
    tau = torch.empty(G * K, dtype=torch.int32, device="cuda")
    mp.mp_ties_tensor_thresholds(L, b, [e] * K, mask, 0.2, tau)
    assert mp.mp_ties_tensor_left() == 0  # the route with lists
    assert torch.equal(tau.view(G, K), one[:, None].expand(G, K))
    held, fixed = mp.mp_workspace_bytes() - before, len(numel) * K * (2048 * 4 + 3 * 16)
    assert held < fixed + (1 << 30), f"{held >> 20} MiB more held after the call"
    mp.mp_release()


def test_repeated_values_overflow_their_lists(mp):  # noqa: F811
    """fp32 deltas of few values, more of them in the bracket than a list holds.
    One value off its bin's floor: the sample leaves at most 512 patterns, a bin
    each, and no pair is left; 127 levels: either way.  Two values with the cut at
    the end of the larger's share: the bracket reaches over both, its lists
    overflow, and the digit passes resolve the bin's open bits of every pair."""
    be, numel = 4096, [300_000, 40_000]
    P, rng = sum(numel), np.random.default_rng(11)
    bits = lambda v: (np.float32(v).view(np.uint32) | np.uint32(1)).view(np.float32)  # noqa: E731
    G = oracle.Blocks(numel, be).G
    base = np.zeros(P, np.float32)
    some = rng.integers(0, 4, G).astype(np.uint32)
    levels = np.clip(np.round(rng.normal(0.0, 30.0, P)), -127, 127) * np.float32(3.3e-5)
    exps = [(bits(1.2345e-3) * rng.choice([-1.0, 0.0, 1.0], P)).astype(np.float32), levels.astype(np.float32)]
    for density in (0.05, 0.2, 0.5, 0.9):
        _say(f"case density {density}")
        _check(mp, "f32", be, numel, base, exps[:1], np.full(G, 1, np.uint32), density)
        assert mp.mp_ties_tensor_left() == 0, mp.mp_ties_tensor_left()
        _check(mp, "f32", be, numel, base, exps, np.full(G, 3, np.uint32), density)
        _check(mp, "f32", be, numel, base, exps, some, density)
        _check(mp, "f32", be, numel, base, exps, some, density, delta=True)
    for one, two in ((bits(2.5e-3), bits(1.2345e-3)), (bits(3.1e-3), bits(3.0e-3))):
        exps = []
        for _ in range(2):
            e = np.zeros(P, np.float32)
            for lo, n in zip(np.cumsum([0] + numel[:-1]), numel):
                # exactly a fifth of the larger, so that the cut is at its end
                v = np.repeat(np.array([one, two, 0.0], np.float32), [n // 5, n // 2, n - n // 5 - n // 2])
                e[lo:lo + n] = rng.permutation(v) * rng.choice([-1.0, 1.0], n).astype(np.float32)
            exps.append(e)
        for density in (0.2, 0.2 + 4 / 300_000):
            _say(f"case two values, density {density}")
            _check(mp, "f32", be, numel, base, exps, np.full(G, 3, np.uint32), density)
            assert mp.mp_ties_tensor_left() == 4, mp.mp_ties_tensor_left()
        _check(mp, "f32", be, numel, base, exps, some, 0.1)
        _check(mp, "f32", be, numel, base, exps, some, 0.1, delta=True)
