"""Grows of small volumes by the schedule they name: the one-block rounds, which
take such volumes whatever the schedule, are switched off (MF4D_ONE_BLOCK=0), so the
launched and the cooperative kernels run at the edge sizes, with one label word a
trajectory and with several.  The tests are those of the other files."""
import pytest

from tests.test_gpu_causal import test_golden_fixtures_forward, test_random_small_ragged_forward  # noqa: F401
from tests.test_gpu_grow_edges import test_edges_match_oracle, test_long_trajectories_match_oracle  # noqa: F401
from tests.test_gpu_grow_read import test_grow_read_over_several_chunks, test_grow_read_round_cap_then_resume  # noqa: F401
from tests.test_gpu_parity import (test_config1, test_golden_fixtures_on_gpu, test_random_small_ragged,  # noqa: F401
                                   test_repeat_grows_identical, test_round_cap_then_resume)
from tests.test_gpu_rate import test_random_rates  # noqa: F401
from tests.test_gpu_submit import test_first_chunk_too_short_and_round_cap  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _no_one_block(monkeypatch):
    monkeypatch.setenv("MF4D_ONE_BLOCK", "0")
