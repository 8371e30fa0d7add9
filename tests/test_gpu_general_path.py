"""Batches of up to 2^19 updates go through buckets, so the tests of rules, shapes and recovery, whose batches are small, see
little of the path of the larger ones: the sort, the chain tiers, and hold-back beside them.  Here the same tests run with
every context's knob set to send its batches there."""
import pytest

from paper_2104_01981_amd import Ecrm
from test_gpu_random_shapes import *        # noqa: F401,F403
from test_gpu_recovery_load import *        # noqa: F401,F403
from test_gpu_recovery_random import *      # noqa: F401,F403
from test_gpu_recovery_read_runs import *   # noqa: F401,F403
from test_gpu_rules import *                # noqa: F401,F403

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def general_path(monkeypatch):
    create = Ecrm.__init__

    def tuned(self, *args, **kwargs):
        create(self, *args, **kwargs)
        self.tune(1, 0xFFFFFFFF)            # ECRM_TUNE_MID_MIN_ROWS

    monkeypatch.setattr(Ecrm, "__init__", tuned)
