"""Workspace of the lag-order selection (host query): no more than the VAR fit's workspace at p_max
plus three m x m matrices and the scratch of a 64-wide panel per lag order."""
import pytest


@pytest.mark.parametrize("m,p,n", [(400, 8, 10000), (400, 1, 10000), (1000, 4, 20000),
                                   (100, 12, 5000), (64, 3, 3000), (10, 10, 1000), (2, 1, 100)])
def test_select_lag_workspace_is_bounded(m, p, n):
    from paper_2409_05500_amd._lib import lib
    var = lib.varlingam_fit_var_workspace_bytes(n, m, p, 1)
    lag = lib.varlingam_select_lag_workspace_bytes(n, m, p)
    panel = 8 * (4096 + 64) if m < 128 else 0
    assert 0 < var and lag <= var + 8 * (3 * m * m) + p * 2 * panel + 4096
