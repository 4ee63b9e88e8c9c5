"""The tuning table's values (no GPU): every candidate can be set and read
back, the number of depth slabs starts as the library's own choice, and that
state can be restored."""
import pytest

from paper_2308_04669_amd import api
from paper_2308_04669_amd._abi import NedfError


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_slabs_automatic_is_no_candidate(dtype):
    old = api.tune_get("slabs", dtype)
    assert old == 0 and old not in api.tune_candidates("slabs", dtype)
    try:
        for v in api.tune_candidates("slabs", dtype):
            api.tune_set("slabs", dtype, v)
            assert api.tune_get("slabs", dtype) == v
        for v in (-1, 3, 64):
            with pytest.raises(NedfError):
                api.tune_set("slabs", dtype, v)
    finally:
        api.tune_set("slabs", dtype, old)
    assert api.tune_get("slabs", dtype) == old


@pytest.mark.parametrize("kernel", ["march", "nedf"])
def test_launch_shapes_have_no_automatic_value(kernel):
    old = api.tune_get(kernel, "bf16")
    assert old in api.tune_candidates(kernel, "bf16")
    with pytest.raises(NedfError):
        api.tune_set(kernel, "bf16", 0)
    assert api.tune_get(kernel, "bf16") == old
