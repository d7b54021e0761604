"""Which calls ask for a workspace (host only).

Single FP32 calls, for the form on the FP16 matrix cores: long sums whose batch one
launch of the FP32 kernel does in less time do not, and neither do short sums, small
outputs and other kernels.  Batch statistics: from the size on that the binding has
from the library itself."""
import pytest

import paper_2110_14502_amd as R


def _need(m, n, k, batch, kernel=-1, shared_b=False):
    M, N, K = list(range(m)), list(range(100, 100 + n)), list(range(200, 200 + k))
    return R.pair_workspace_bytes(K + M, N + K, M + N, kernel=kernel, batch=batch, stride_a=1 << (m + k),
                                  stride_b=0 if shared_b else 1 << (n + k))


@pytest.mark.parametrize("m,n,k,batch,taken", [
    (8, 7, 10, 1, True), (8, 7, 10, 2, True), (8, 7, 10, 32, False), (8, 7, 10, 64, False), (9, 8, 10, 32, False),
    (8, 7, 13, 32, False), (12, 12, 12, 1, True), (12, 12, 12, 8, True), (12, 12, 12, 65, False), (7, 7, 12, 1, False),
    (12, 12, 7, 1, False), (13, 13, 8, 1, True)])
def test_batches_of_long_sums(m, n, k, batch, taken):
    need = _need(m, n, k, batch)
    assert (need >= 12 * batch * ((1 << (m + k)) + (1 << (n + k)))) == taken
    assert need == _need(n, m, k, batch)  # exchanged operands
    assert _need(m, n, k, batch, kernel=1) == 0


def test_batch_statistics_threshold():
    n = R._XEB_SPLIT
    assert R._xeb_workspace(n, 0) and R._xeb_workspace(0, n) and not R._xeb_workspace(n - 1, n - 1)
