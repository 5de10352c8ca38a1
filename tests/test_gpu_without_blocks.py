"""The tests of the sweep, of the single launch for small graphs and of the
multi-kernel hand-over on graphs that one block per column solves by default:
here with that solver off (NVD_COLUMN=0), so that they run what they name."""
import pytest

from test_gpu_batch import (test_small_batch_matches_oracle, test_tiles_across_widths,            # noqa: F401
                            test_uneven_k_and_equivalence_with_single_solves)
from test_gpu_refine import test_guard_quiet_on_well_conditioned_graph, test_stalled_pairs_are_finished_in_fp64  # noqa: F401
from test_gpu_small import (test_mid_path_noconv_and_forced_handover, test_mid_path_repeatable_degenerate_and_dsq,  # noqa: F401
                            test_small_path_c1_and_repeatable, test_small_path_degenerate_and_noconv,
                            test_small_path_forced_fp64_handover,
                            test_small_path_matches_oracle_and_multikernel)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _no_blocks(monkeypatch):
    monkeypatch.setenv("NVD_COLUMN", "0")
