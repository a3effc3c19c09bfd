"""Error of the runtime-radix transforms: every pass twiddle is one product of
two table entries.  The bounds are the
errors on the same inputs of the transforms by sevens, fives, nines and radices
16, 8, 4 and 2 (the same twiddles; 8 x 8 x 8 is 16 x 16 x 2 there) and 1%."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import run_plan, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,err", [(49, 8.2438e-8), (343, 1.1072e-7), (729, 1.3118e-7),
                                   (1715, 1.2842e-7), (2401, 1.3140e-7), (6561, 1.5389e-7),
                                   (12005, 1.4710e-7), (59049, 2.0258e-7), (1835008, 2.1389e-7),
                                   # radices of 10 and more in most passes
                                   (3136, 1.2844e-7), (5000, 1.3916e-7), (6272, 1.3602e-7),
                                   (7000, 1.3845e-7), (10000, 1.4098e-7), (15625, 1.5857e-7)])
def test_error(n, err):
    import paper_1203_4938_amd as dp
    batch = max(1, (1 << 17) // n)
    x = synth.uniform_complex(synth.BASE_SEED + 890, n, batch)
    y = run_plan(dp.Plan(n, batch), to_dev(x)).cpu().numpy()
    ref = oracle.fft_batch(x)
    e = float(np.linalg.norm(y - ref) / np.linalg.norm(ref))
    say(f"[mixed error] {n}: {e:.4e} of {err:.4e}, {e / err:.3f}")
    assert e <= 1.01 * err
