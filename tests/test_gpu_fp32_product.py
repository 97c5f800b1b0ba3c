"""The FP32 rotation product (DE_GEMM_FP32) through the C ABI: values that
depend on the row and R alone.
"""
import pytest

from tests import test_gpu_kernel_edges as edges

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    yield


# run 0 of a handle of one run equals run 0 of a handle of many, and the value
# of a row does not depend on how many rows are evaluated with it, at the
# widths of 513 to 1024 coordinates too
@pytest.mark.parametrize("NP,D,many,jde", [
    (33, 513, 130, None), (65, 640, 90, True), (64, 700, 129, None),
    (97, 769, 70, None), (33, 1000, 130, None), (40, 1024, 129, True),
])
def test_values_do_not_depend_on_the_number_of_runs(NP, D, many, jde):
    edges.test_few_tiles_equal_many("fp32", NP, D, many, jde)
