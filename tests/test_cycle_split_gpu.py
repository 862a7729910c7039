"""Cycle-scan over the numbers of waves that share a chunk's states: the launch picks them by the
number of (batch entry, chunk, 64 channels) groups, so many short batch entries reach every
instance with little data.  Remainders: 1, 2 and 3 tokens past the groups of four, one live lane.
The bound is that of the parity tests: max|y - y_oracle| <= (4 * 2^-24 / min|Delta a| + 1e-6)
max|y_oracle|, from the absolute error 2^-24 of the hardware exp2 near 1."""
import numpy as np
import pytest
import torch

from oracle import cycle_scan as CS
from paper_2407_02109_amd import binding as fb, synth

pytestmark = pytest.mark.gpu

CASES = [  # B, L, d, N
    # waves per group in pass A / C: 8/8 | 4/4, 4/4 | 4/1
    (1023, 5, 1, 32), (1024, 6, 3, 32), (2815, 7, 2, 32), (2816, 5, 1, 32), (3071, 7, 2, 32), (3072, 5, 3, 32),
    # 4/4 | 2/1, 2/1 | 1/1, 1/1 | 1/1 early, early | 1/1
    (1536, 5, 1, 16), (1537, 6, 2, 16), (2047, 3, 2, 16), (2048, 7, 1, 16), (3072, 6, 2, 16), (3073, 7, 3, 16),
    (5120, 5, 2, 16), (5121, 7, 1, 16), (6143, 6, 2, 16), (6144, 5, 1, 16), (6145, 7, 2, 16), (2561, 35, 66, 16),
    (3072, 35, 65, 32), (40, 35, 65, 32),   # two chunks, two channel groups
    (64, 9, 70, 8), (64, 9, 70, 4),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_split_instances(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, L, d, N = case
    print("[case] cycle split %s" % (case,), flush=True)
    x, delta, A, Bm, Cm = synth.make_cycle_inputs(B, L, d, N, seed=B + N, kind="wide")
    out = torch.full((B, L, d), float("nan"), device="cuda")
    y = fb.cycle_scan(*(t.to("cuda") for t in (x, delta, A, Bm, Cm)), repeats=3, out=out).cpu().double().numpy()
    pick = sorted({0, 1, B // 2, B - 1})   # batch entries checked against the definition
    ref = CS.cycle_scan(*(t[pick].double().numpy() for t in (x, delta)), A.double().numpy(),
                        *(t[pick].double().numpy() for t in (Bm, Cm)), 3)
    assert np.isfinite(y).all()
    m = (delta.abs().amin(dim=(0, 1))[:, None] * A.abs()).min().item()
    assert np.abs(y[pick] - ref).max() <= (4.0 * 2.0 ** -24 / m + 1e-6) * np.abs(ref).max()
