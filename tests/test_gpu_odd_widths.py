"""Steps on rows of no whole 16 bytes, the narrowest included: the chain rule reads such rows 16 bytes at a time from any multiple of 4
bytes, their last columns with those before them."""
import pytest

from parity_util import run_step_both, check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", (2, 3, 5, 6, 7, 63, 66, 131, 255, 258, 399))
def test_one_step(dim):
    # (rows of one column are left out: a row is then one sum of terms of either sign, whose rounding has no bound against the sum)
    for model, B, C, N in ((0, 90, 3, 40), (2, 90, 3, 40), (3, 700, 2, 300)):
        print("case", dim, model, flush=True)
        print(check_step(run_step_both(model, 500, 4, dim, B, C, N, B - 11, seed=dim, std=0.3)), flush=True)
