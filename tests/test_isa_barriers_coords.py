"""The barrier check of tests/test_isa_barriers.py on the pair solver's
second translation unit (the variants with coordinates in LDS)."""
import os
import shutil

import pytest

from tests import test_isa_barriers as base


@pytest.mark.skipif(not shutil.which(base.HIPCC) and not os.path.exists(base.HIPCC), reason="hipcc not available")
def test_coordinate_variants(tmp_path):
    base.test_solver_kernels_have_no_divergent_back_edge_into_a_barrier(tmp_path, "pair_solver_coords.hip")
