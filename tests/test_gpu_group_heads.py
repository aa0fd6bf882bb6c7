"""Group decode at the query-head counts where its kernels change: one and two head tiles on
the matrix cores (16 | 17 and 32 heads per group), every group size, lengths on both sides of
the 256-token splits and several splits into one merge.  Same bar as the other group tests:
records and scales bit-exact, outputs within 2e-3 relative L2 of the oracle."""
import pytest

from test_gpu_groups import GCase, _run

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("gkv,heads,groups", [(1, 16, 2), (1, 17, 2), (1, 32, 1), (2, 18, 1), (2, 32, 1),
                                              (3, 21, 1), (4, 20, 2), (4, 32, 1)])
def test_heads_per_group(gkv, heads, groups):
    case = GCase(2, gkv, [0, 1, 256, 257, 1100], n_kv_heads=gkv * groups, n_q_heads=heads * groups)
    _run(case)
