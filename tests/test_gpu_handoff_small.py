"""The hand-off selection where more literals are asked for than there are
variables: the sort runs over the variables' power of two."""
import pytest

from paper_2511_07737_amd import tsat

import test_gpu_handoff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,k", [(3, 1), (3, 2), (3, 4096), (251, 255), (251, 256), (251, 257), (252, 4096), (600, 4096)])
def test_more_literals_than_variables(V, k):
    test_gpu_handoff.test_selection_equals_host_ranking(V, 4 * V, 3, 40, 5, k, 1.0, tsat.MODE_NONE)
