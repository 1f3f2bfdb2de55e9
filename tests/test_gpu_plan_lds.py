"""The planner's two ways of reading the grouping arrays, from LDS (up to 1023 groups and 4096 members) and from
memory (more), give the same plan.

Empty groups and empty members add no work, so a problem just inside the line and the same problem with one more
of them, just outside it, must give bitwise-identical outputs and gradients.
"""
import numpy as np
import pytest

from paper_2506_05433_amd.inputs import make_problem
from tests._parity import GRADS, OUTS, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NAMES = ("q_pre", "k_pre", "v_pre", "q_suf", "k_suf", "v_suf")


def _lengths(groups, members, seed):
    """`groups` groups that share `members` members, every length ragged and some of them 0."""
    rng = np.random.default_rng(seed)
    sizes = np.bincount(rng.integers(0, groups, members), minlength=groups)
    return tuple(rng.integers(0, 8, groups)), tuple(sizes), tuple(rng.integers(0, 5, members))


def _run(lengths, dtype):
    from paper_2506_05433_amd import binding
    prob = make_problem("single_group", seed=730, lengths=lengths, h_q=4, h_kv=2, head_dim=64, dtype=dtype,
                        scale=0.125)
    dev = binding.to_device(prob, "cuda")
    f = binding.run_fwd(dev)
    out = dict(zip(OUTS, f))
    out.update(zip(GRADS, binding.run_bwd(dev, f)))
    o, lse = binding.fwd_last(*[dev[n] for n in NAMES], dev["cu_prefix"], dev["cu_suffix"], dev["group_sizes"],
                              dev["scale"])
    torch.cuda.synchronize()
    m = len(lengths[2]) if lengths[2][-1] else len(lengths[2]) - 1
    out.update(last_o=o[:m], last_lse=lse[:, :m])
    return {k: to_host(v) for k, v in out.items()}


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("line", ["groups", "members"])
def test_plan_from_lds_matches_plan_from_memory(line, dtype):
    print(f"[plan lds] {line} {dtype}", flush=True)
    if line == "groups":
        p, g, s = _lengths(1023, 300, 1)
        inside, outside = (p, g, s[:-1] + (3,)), (p + (0,), g + (0,), s[:-1] + (3,))
    else:
        p, g, s = _lengths(700, 4096, 2)
        s = s[:-1] + (3,)
        inside, outside = (p, g, s), (p, g[:-1] + (g[-1] + 1,), s + (0,))
    a, b = _run(inside, dtype), _run(outside, dtype)
    assert a["o_pre"].shape == b["o_pre"].shape and np.isfinite(a["o_suf"]).all()
    for k in a:
        assert np.array_equal(a[k], b[k]), f"{k}: the two plans gave different results"


def _plan_us(call):
    from paper_2506_05433_amd import binding
    best = float("inf")
    for _ in range(3):
        torch.cuda.synchronize()
        binding.timing_start()
        for _ in range(10):
            call()
        torch.cuda.synchronize()
        binding.timing_stop()
        n, ms = binding.timing_get("plan")
        best = min(best, ms / n * 1e3)
    return best


def test_planning_from_lds_is_no_slower_than_from_memory():
    """At its largest size, where sums that walk all groups in every thread took 93 us (8.6 us with scans, 11.5 us
    from memory)."""
    from paper_2506_05433_amd import binding
    p, g, s = _lengths(1023, 1023, 3)
    times = []
    for lengths in ((p, g, s), (p + (0,), g + (0,), s)):
        dev = binding.to_device(make_problem("single_group", seed=731, lengths=lengths, h_q=2, h_kv=2, head_dim=64), "cuda")
        args = (dev["q_pre"], dev["q_suf"], dev["k_pre"], dev["k_suf"], dev["cu_prefix"], dev["cu_suffix"],
                dev["group_sizes"])
        times.append(_plan_us(lambda: binding.rope(*args)))
    print(f"[plan lds] inside {times[0]:.1f} us, outside {times[1]:.1f} us", flush=True)
    assert times[0] <= 1.5 * times[1], times
