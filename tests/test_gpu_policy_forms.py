"""The three forms of the fused policy kernel (16, 32 or 64 environments per
wave, chosen by batch size) and the corners of its weight tables: the forms give
the same bits, weights may sit at any address their own type allows, and
non-finite hidden-layer weights mean what fp32 arithmetic makes of them."""
import numpy as np
import pytest

import workloads
from gpu_helpers import device_policy, policy_weights

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PLANES = ("obs", "action", "reward", "done", "policy_p0", "logp", "value")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(n, K, calls, w, dtype, seed, env0=0, tens=None):
    """Trajectory planes and per-call statistics of `calls` launches of K steps."""
    import paper_2207_07736_amd as p
    st, keep = device_policy(w, dtype)
    if tens is not None:
        st, keep = tens
    sim = p.Simulator(n, 0, workloads.CARTPOLE, env0=env0)
    try:
        sim.reset(seed)
        tr = p.Trajectory(K * calls, n, p0=True, learner=True)
        stats = []
        for c in range(calls):
            sim.step(K, tr.rows(c * K, K), policy=st)
            stats.append(tr.block_stats.cpu().numpy())
        out = {k: getattr(tr, k).cpu().numpy() for k in PLANES}
        out["state"], out["ep"], _ = sim.get_state()
        del keep
        return out, np.stack(stats)
    finally:
        sim.close()


def _same(a, b):
    return np.array_equal(a.view(np.uint32) if a.dtype == np.float32 else a,
                          b.view(np.uint32) if b.dtype == np.float32 else b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sizes", [(49152, 98304 - 49152 + 300), (768, 50176, 49152 + 63)])
def test_forms_agree_bit_for_bit(dtype, sizes):
    """One batch of 98,305 or more environments (64 per wave) against shards of
    it in the smaller forms: 49,152 is the last size with 16 per wave, sizes up
    to 98,304 run 32 (fp32) or 64 (bf16); ragged last blocks among them."""
    w, K, calls, seed = policy_weights(21, 0.3), 9, 3, 3
    n = sum(sizes)
    assert n > 98304
    whole, stats = _run(n, K, calls, w, dtype, seed)
    assert stats[-1].sum() > 0
    at = 0
    for size in sizes:
        part, part_stats = _run(size, K, calls, w, dtype, seed, env0=at)
        for k in PLANES + ("state", "ep"):
            assert _same(part[k], np.ascontiguousarray(whole[k][..., at:at + size])), (k, size)
        if size % 256 == 0:
            assert np.array_equal(part_stats, stats[:, at // 256:(at + size) // 256]), size
        else:
            assert np.array_equal(part_stats, stats[:, at // 256:]), size
        at += size


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [1, 3])
def test_weights_at_any_element_address(dtype, shift):
    """Weights that start `shift` elements into an allocation give what aligned
    ones give (the ABI asks for the weight's own alignment only)."""
    import paper_2207_07736_amd as p
    w = policy_weights(5, 0.3)
    st, tens = device_policy(w, dtype)
    moved = dict(tens)
    for k in ("w1", "w2", "w3", "wv"):
        buf = torch.zeros(tens[k].numel() + shift, dtype=tens[k].dtype, device="cuda")
        buf[shift:] = tens[k].reshape(-1)
        moved[k] = buf[shift:]
    st2 = p.policy_struct(p.RLSIM_BF16 if dtype == "bf16" else p.RLSIM_F32, moved["w1"], moved["b1"], moved["w2"],
                          moved["b2"], moved["w3"], moved["b3"], moved["wv"], moved["bv"])
    a, _ = _run(300, 5, 2, w, dtype, 1)
    b, _ = _run(300, 5, 2, w, dtype, 1, tens=(st2, moved))
    for k in PLANES:
        assert _same(a[k], b[k]), k


@pytest.mark.parametrize("n", [300, 50000, 98560])
def test_fp32_hidden_weights_that_are_not_finite(n):
    """An infinite W2 entry saturates its unit to the sign of its input, a NaN one
    makes every output NaN (action 1), as in plain fp32 arithmetic.  The reference
    is 64-bit; fp32 sums of 64 terms below 1 in magnitude are within
    64 * 2^-24 = 4e-6 of it."""
    w = policy_weights(9, 0.3)
    w["w2"] = w["w2"].copy()
    w["w2"][3, 17], w["w2"][40, 2], w["w2"][11, 60] = np.inf, -np.inf, 3.0e38
    out, _ = _run(n, 1, 1, w, "f32", 2)
    obs = out["obs"][0].T.astype(np.float64)
    f = {k: v.astype(np.float64) for k, v in w.items()}
    h1 = np.tanh(obs @ f["w1"].T + f["b1"])
    z = np.stack([(h1 * f["w2"][r]).sum(1) for r in range(64)], 1) + f["b2"]
    h2 = np.tanh(z)
    logit = h2 @ f["w3"].T + f["b3"]
    p0 = 1.0 / (1.0 + np.exp(logit[:, 1] - logit[:, 0]))
    assert np.all(np.isfinite(p0))
    assert np.max(np.abs(out["policy_p0"][0] - p0)) <= 4e-6
    assert np.max(np.abs(out["value"][0] - (h2 @ f["wv"].T + f["bv"])[:, 0])) <= 3e-5
    w["w2"][50, 50] = np.nan
    out, _ = _run(n, 1, 1, w, "f32", 2)
    assert np.all(np.isnan(out["policy_p0"])) and np.all(np.isnan(out["value"])) and np.all(out["action"] == 1)


FLT_MAX = np.finfo(np.float32).max


@pytest.mark.parametrize("large", [np.inf, FLT_MAX])
def test_forms_agree_bit_for_bit_on_the_plain_layer(large):
    """One W2 entry that the split layer does not take: its unit saturates, and
    the finite units keep the same bits in every form."""
    w, K, seed = policy_weights(21, 0.3), 9, 3
    w["w2"] = w["w2"].copy()
    w["w2"][3, 17] = large
    whole, _ = _run(98560, K, 1, w, "f32", seed)            # 64 per wave
    for env0, size in ((0, 49152), (98304, 67), (256, 49153), (0, 98304)):      # 16, 16, 32, 32
        part, _ = _run(size, K, 1, w, "f32", seed, env0=env0)
        for k in PLANES + ("state", "ep"):
            assert _same(part[k], np.ascontiguousarray(whole[k][..., env0:env0 + size])), (k, env0, size)


@pytest.mark.parametrize("n", [300, 50000, 98560])
@pytest.mark.parametrize("entries", [
    [(40, 2, -FLT_MAX)], [(11, 60, 3.397e38)],      # infinite when rounded to bfloat16
    [(5, 33, 3.38e38), (5, 34, -1.0e37)]])          # finite in bfloat16 too
def test_fp32_hidden_weights_that_are_very_large(n, entries):
    """A very large finite W2 entry saturates its unit to the sign of its input
    and every output stays finite, with no infinity among the weights."""
    w = policy_weights(9, 0.3)
    w["w2"] = w["w2"].copy()
    for r, c, v in entries:
        w["w2"][r, c] = v
    _against_64_bits(n, w)


@pytest.mark.parametrize("n", [300, 50000, 98560])
def test_fp32_large_hidden_weights_that_cancel(n):
    """Eight weights of 3e38 against eight of -3e38 on saturated units: added one
    unit of each at a time they cancel, where the sum of either eight overflows."""
    w = policy_weights(9, 0.3)
    w["w1"], w["b1"], w["w2"], w["b2"] = (w[k].copy() for k in ("w1", "b1", "w2", "b2"))
    w["w1"][:16], w["b1"][:16] = 0.0, 20.0              # h1 = 1 exactly
    plus = [0, 1, 2, 3, 8, 9, 10, 11]
    w["w2"][7], w["b2"][7] = 0.0, 0.0
    w["w2"][7, :16] = -3.0e38
    w["w2"][7, plus] = 3.0e38
    _against_64_bits(n, w)


def _against_64_bits(n, w):
    """One step against the network in 64 bits.  fp32 sums of 64 terms below 1 in
    magnitude are within 64 * 2^-24 = 4e-6 of it."""
    out, _ = _run(n, 1, 1, w, "f32", 2)
    obs = out["obs"][0].T.astype(np.float64)
    f = {k: v.astype(np.float64) for k, v in w.items()}
    h1 = np.tanh(obs @ f["w1"].T + f["b1"])
    h2 = np.tanh(np.stack([(h1 * f["w2"][r]).sum(1) for r in range(64)], 1) + f["b2"])
    logit = h2 @ f["w3"].T + f["b3"]
    p0 = 1.0 / (1.0 + np.exp(logit[:, 1] - logit[:, 0]))
    assert np.all(np.isfinite(p0))
    assert np.max(np.abs(out["policy_p0"][0] - p0)) <= 4e-6
    assert np.max(np.abs(out["value"][0] - (h2 @ f["wv"].T + f["bv"])[:, 0])) <= 3e-5


@pytest.mark.parametrize("n", [256, 50176, 98560])
def test_fp32_hidden_products_are_whole(n):
    """One hidden weight per row and a bias that cancels most of the product:
    the fp32 layer keeps every bit of both factors.  What is left out of a product
    is below 2^-34 of it, and its small parts (within 2^-7 of it) are summed in
    eight fp32 additions: 8 * 2^-24 * 2^-7 = 2^-28 together.  The sum of its
    leading part and the bias is exact where they cancel.  S = 2^12 shows 2^-28 of
    a product as 1.5e-5 to 3e-5 of the unit's input, against 1.3e-6 that its tanh
    (2.5e-7, through a slope of 0.19 or more) hides.  Three of the nine products of
    the bfloat16 pieces left out, or all summed on the bias, show as 2^-24 and more."""
    S = 4096.0
    rng = np.random.default_rng(0)
    for unit in range(0, 64, 7):
        c = np.float32(np.arctanh(rng.uniform(0.55, 0.95)))
        centre = np.tanh(np.float64(c))
        # the unit's exact h1, read through a weight that is a power of two
        b = np.float64(np.float32(S * centre))
        z = _one_unit(n, unit, c, S, b)
        x = np.rint((z + b) * 4096.0) / 4096.0 / S      # h1 >= 0.5 is a multiple of 2^-24
        for w in (1.0038986, 1.0 + 2.0 ** -8 - 2.0 ** -17, rng.uniform(1.0, 2.0)):
            w = np.float64(np.float32(S * w))
            b = np.float64(np.float32(w * centre))
            got = _one_unit(n, unit, c, w, b)
            use = (np.abs(z) < 1.4) & (np.abs(got) < 1.4)
            assert use.sum() > n // 4
            err = np.abs(got - (w * x - b))[use]
            assert np.all(err <= 2.0 ** -28 * w * x[use] + 2.0e-6), (unit, w, err.max())


def _one_unit(n, unit, c, weight, minus_bias):
    """Layer-2 input of hidden unit `unit` for n environments whose h1 there is
    tanh(c + 0.002 x) and its only weight `weight`."""
    zero = dict(w1=(64, 4), b1=64, w2=(64, 64), b2=64, w3=(2, 64), b3=2, wv=(1, 64), bv=1)
    w = {k: np.zeros(v, dtype=np.float32) for k, v in zero.items()}
    w["w1"][unit, 0], w["b1"][unit] = 0.002, c
    w["w2"][unit, unit], w["b2"][unit], w["wv"][0, unit] = weight, -minus_bias, 1.0
    out, _ = _run(n, 1, 1, w, "f32", 3)
    return np.arctanh(np.clip(out["value"][0].astype(np.float64), -1.0 + 1e-9, 1.0 - 1e-9))
