"""The inline asm of the split kernel's small-call instances against the MFMA
wait-state rules, as tests/test_asm_hazards.py does for the other instances (CPU only:
hipcc)."""
import os
import shutil

import pytest

from test_asm_hazards import test_inline_asm_respects_mfma_wait_states as _scan_unit


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not installed")
def test_team_instances_respect_mfma_wait_states(tmp_path):
    _scan_unit(tmp_path, "decode_mfma_team.hip")
