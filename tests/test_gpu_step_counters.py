"""The tests of the persistent kernels that order their steps by counters, or run one layer per launch, once more without the kernels of
16-row slices, which take many of these shapes since they came (LSTM_NEAR=0: also what devices with fewer CUs run)."""
import pytest

from test_gpu_granular_hidden import test_narrow, test_other_cells, test_scratch_line_of_many_workgroups  # noqa: F401
from test_gpu_large_mid import test_long_products, test_padded  # noqa: F401
from test_gpu_large_mid import test_other_cells as test_one_layer_kernels_of_other_cells  # noqa: F401
from test_gpu_parity import test_persistent_layer_groups, test_persistent_shapes, test_persistent_variants  # noqa: F401
from test_gpu_rnn_cells import test_large_hidden_shapes, test_measured_shape_at_full_size  # noqa: F401
from test_gpu_rnn_cells import test_persistent_layer_groups as test_layer_groups_of_other_cells  # noqa: F401
from test_gpu_rnn_cells import test_persistent_shapes as test_shapes_of_other_cells  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def step_counters(knobs):
    knobs(LSTM_NEAR="0")
