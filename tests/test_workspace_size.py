"""Workspace bytes of 1-D problems (no GPU needed).  A caller may keep an arena of a
fixed size, and the allocation-free entry point does: the size follows from the
problem's arrays and one work item per 256 replicas of a window, whatever the
number of lanes a replica gets."""
import pytest

import paper_1105_4840_amd as ppp
import ppp_inputs


def _size(replicas, windows, **kw):
    p = ppp_inputs.config_1d(n_replicas=replicas, n_windows=windows)
    p.update(kw)
    h = ppp.ppp_create(p)
    try:
        return ppp.ppp_workspace_size(h)
    finally:
        ppp.ppp_destroy(h)


# sizes with one lane a replica
@pytest.mark.parametrize("replicas,windows,plain,free,sequential,fp32", [
    (256, 21, 20150272, 20224000, 20150016, 20107264),
    (195, 21, 19965952, 20030976, 19965696, 19933184),
    (16, 5, 4613632, 4650752, 4613632, 4613120),
    (256, 4, 3841024, 3915008, 3841024, 3832832),
    (4096, 2, 3028480, 3655680, 3028224, 2962944),
    (65, 690, 642998016, 643044608, 642987008, 642639104),
    (3000, 21, 28451840, 28920832, 28448000, 27947776),
])
def test_size_does_not_depend_on_the_lanes(replicas, windows, plain, free, sequential, fp32):
    assert _size(replicas, windows) == plain
    assert _size(replicas, windows, free_ensemble=True) == free
    assert _size(replicas, windows, sequential=True) == sequential
    assert _size(replicas, windows, precision="fp32") == fp32


@pytest.mark.parametrize("replicas,windows,bins", [(195, 21, 395192), (37, 100, 82480)])
def test_largest_problems_of_the_static_workspace_fit(replicas, windows, bins):
    kw = dict(w_half_bins=0)
    assert _size(replicas, windows, xi_nbins=bins, **kw) <= ppp.PPP_STATIC_WORKSPACE_BYTES
    assert _size(replicas, windows, xi_nbins=bins + 16, **kw) > ppp.PPP_STATIC_WORKSPACE_BYTES
