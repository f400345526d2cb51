"""Workgroups of the default adjoint (no GPU): windows that no output row of a
block lies in are not launched, so a smallest delay, or delays longer than the
record, do not multiply the work."""
import pytest

torch = pytest.importorskip("torch")

import paper_1411_5373_amd as F  # noqa: E402


def _items(nf, nt, nd, **kw):
    return [s["work_items"] for s in F.Plan(nf, nt, nd, 1.2, 1.6, host_only=True, **kw).steps(True)]


@pytest.mark.parametrize("nf,nt,nd", [(1024, 1024, 64), (64, 1024, 64), (64, 20000, 64), (1000, 3000, 200)])
@pytest.mark.parametrize("d_min", (300, 10000, 100000))
def test_smallest_delay(nf, nt, nd, d_min):
    """The last pass applies the delay: at most a channel's own spread more."""
    plain, late = _items(nf, nt, nd), _items(nf, nt, nd, d_min=d_min)
    if len(late) == len(plain):
        assert late[:-1] == plain[:-1]
        assert late[-1] <= 8 * plain[-1]
    assert sum(late) <= 8 * sum(plain)


@pytest.mark.parametrize("nf,nt,nd", [(1024, 512, 2048), (2048, 300, 1900), (256, 100, 2000)])
def test_delays_longer_than_the_record(nf, nt, nd):
    """The first pass shifts by up to the delay: less than twice its rows' windows."""
    items = _items(nf, nt, nd)
    assert items[0] <= 2 * ((nd + 6) // 7) * (nt // 224 + 2)
