"""The per-call state pointers: null pointers in any form through the binding."""
import numpy as np
import pytest

import paper_2411_19379_amd as ssm
from paper_2411_19379_amd import binding


@pytest.mark.parametrize("nulls", [[None, None], [0, None], np.zeros(2, np.int64), (False, 0.0)])
def test_null_pointers_in_any_form(nulls):
    plan = ssm.Plan(4, 16, 16, 1, 64, "f32", [0, 3, 5], None)
    assert list(binding._ptr_array(plan.handle, nulls)) == [None, None]
    assert list(binding._ptr_array(plan.handle, [0, 4096])) == [None, 4096]
    plan.close()
