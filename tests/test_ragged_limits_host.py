"""Longest beam of a ragged batch: the kernels index samples, their shifts and
their tiles in 32 bits, so a beam that leaves no room for these below 2^31 is
refused before any device work (a host-only plan is refused last)."""
import pytest

torch = pytest.importorskip("torch")

import paper_1411_5373_amd as F  # noqa: E402
from paper_1411_5373_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("nd,d_min,options", [
    (64, 0, {}), (64, 1 << 30, {}), (64, 5000, {"gather_rows": 1, "gather_vecs": 4}), (2048, 0, {"adjoint_levels": 2}),
    (16, 0, {"first_kernel": 2, "tile": 8192, "stream_tiles": 65535}), (65536, 77, {"unfused": True})])
def test_longest_beam(nd, d_min, options):
    plan = F.Plan(32, 1000, nd, 1.2, 1.6, d_min=d_min, host_only=True, **options)
    longest = 2 ** 31 - 1 - d_min - 2 * nd  # less the widest tile and 2^13
    for nt, status, text in ((2 ** 31 - 64, B.FDMT_E_INVALID, "beam 1"), (longest - 8192, B.FDMT_E_INVALID, "beam 1"),
                             (longest - 2 ** 30, B.FDMT_E_UNSUPPORTED, "HOST_ONLY")):
        if nt < 0:
            continue
        with pytest.raises(F.FDMTError) as e:
            B.fdmt_ragged_plan(plan.handle, [0, nt])
        assert e.value.status == status and text in F.fdmt_last_error(), (nt, F.fdmt_last_error())
