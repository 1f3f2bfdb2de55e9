"""GPU parity of the backward's 256-key dK/dV and 256-row dQ kernels at the edges of their tiles.

The sizes are large enough for the library to choose them (test_wide_codegen.py checks the choice) and
ragged everywhere: prefixes one row past a key tile, responses shorter than a query tile, a key tile spanning
several members, empty responses and prefixes, a group without members, GQA ratios 1 to 8, both head dims and both
layouts, with response rows before a prefix in the single buffer. Tolerances are those of every bf16 parity test
(tests/_parity.py).
"""
import numpy as np
import pytest

from paper_2506_05433_amd.inputs import make_problem
from tests.test_gpu_parity import _full_compare
from tests.test_gpu_xours import _run_both

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RAGGED = (1, 33, 0, 700, 256, 511, 64, 31, 400, 90)
CASES = [
    # (lengths, h_q, h_kv, d, kv head compared)
    (((1025,), (10,), RAGGED), 64, 8, 128, 5),
    (((1025,), (10,), RAGGED), 64, 8, 64, 2),
    (((1500, 1100), (10, 0), RAGGED), 64, 8, 128, 7),
    (((1281, 1024), (3, 10), (257, 1, 3200) + RAGGED), 32, 32, 64, 31),
    # response rows before a prefix (a prefix offset in the single buffer), an empty prefix beside a long one
    (((1100, 1300), (4, 6), RAGGED), 64, 8, 64, 4),
    (((2100, 0, 1200), (3, 4, 3), RAGGED), 64, 8, 128, 1),
    # one head: too few tiles to fill the CUs, so each member's rows are tiled on their own
    (((16380,), (5,), (3000, 1, 700, 2491, 2000)), 1, 1, 64, 0),
]

# the dQ kernel as well: prefixes of 8192 rows and more
DQ_CASES = [
    (((8193,), (10,), RAGGED), 16, 16, 128, 3),
    (((8192, 8479), (0, 11), (5,) + RAGGED), 16, 8, 128, 6),
    (((8193, 8479), (4, 7), (5,) + RAGGED), 16, 8, 128, 2),
]


@pytest.mark.parametrize("case", range(len(CASES) + len(DQ_CASES)))
def test_wide_backward(case):
    lengths, hq, hkv, d, kv = (CASES + DQ_CASES)[case]
    prob = make_problem("single_group", seed=700 + case, lengths=lengths, h_q=hq, h_kv=hkv, head_dim=d,
                        scale=1.0 / np.sqrt(d))
    r = hq // hkv
    _full_compare(prob, heads=list(range(kv * r, (kv + 1) * r)), kv_heads=[kv])


@pytest.mark.parametrize("which", [CASES[0], DQ_CASES[1]], ids=["dkdv", "dq"])
def test_wide_backward_with_peaked_softmax(which):
    """Q x 4: sharp rows, whose dP - Dsum is small beside the Dsum that dP starts at."""
    lengths, hq, hkv, d, kv = which
    r = hq // hkv
    prob = make_problem("single_group", seed=705, lengths=lengths, h_q=hq, h_kv=hkv, head_dim=d, peaked=True)
    _full_compare(prob, heads=list(range(kv * r, (kv + 1) * r)), kv_heads=[kv])


@pytest.mark.parametrize("which", [CASES[0], CASES[4], CASES[5], DQ_CASES[1], DQ_CASES[2]],
                         ids=["dkdv", "dkdv_offset_d64", "dkdv_empty_prefix", "dq", "dq_offset"])
def test_wide_backward_xours_and_repeat(which):
    lengths, hq, hkv, d, _ = which
    prob = make_problem("single_group", seed=710, lengths=lengths, h_q=hq, h_kv=hkv, head_dim=d)
    a, _ = _run_both(prob)
    b, _ = _run_both(prob)
    for n in a:
        assert torch.equal(a[n], b[n]), f"{n} differs between two runs"


@pytest.mark.parametrize("d", [64, 128])
def test_nan_query_row_leaves_dv_of_keys_it_does_not_see(d):
    """A key's dV is a sum over the rows that see it: a row whose log-sum-exp is NaN changes no other key's. Rows
    inside a key tile on both sides, so that the tile's mask has to keep them apart."""
    from paper_2506_05433_amd import binding
    lengths, hq, hkv, _, _ = CASES[0]
    prob = make_problem("single_group", seed=720, lengths=lengths, h_q=hq, h_kv=hkv, head_dim=d)
    dev = binding.to_device(prob, "cuda")
    clean = binding.run_bwd(dev, binding.run_fwd(dev))
    starts = np.concatenate([[0], np.cumsum(lengths[2])])
    pre, suf = 1000, int(starts[6]) - 1  # the last row of member 5
    dev["q_pre"][pre] = float("nan")
    dev["q_suf"][suf] = float("nan")
    got = binding.run_bwd(dev, binding.run_fwd(dev))
    torch.cuda.synchronize()
    dv_pre, dv_suf = got[2], got[5]
    # every prefix key is seen by the response row, every key up to its own by a row of its own side
    assert torch.isnan(dv_pre).all() and torch.isnan(dv_suf[int(starts[5]):suf + 1]).all()
    others = [r for r in range(int(starts[-1])) if not int(starts[5]) <= r <= suf]
    assert torch.equal(dv_suf[others], clean[5][others])
    dev["q_suf"][suf] = 0.5  # now only the prefix row is NaN
    f = binding.run_fwd(dev)
    got = binding.run_bwd(dev, f)[2]
    dev["q_pre"][pre] = 0.25
    want = binding.run_bwd(dev, binding.run_fwd(dev))[2]
    torch.cuda.synchronize()
    assert torch.isnan(got[:pre + 1]).all() and torch.equal(got[pre + 1:], want[pre + 1:])
