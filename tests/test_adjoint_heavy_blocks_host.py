"""Blocks of the default adjoint (no GPU) under wide sub-bands: ranges whose rows
read many more rows of the plane above than the others are split further."""
import pytest

torch = pytest.importorskip("torch")

import paper_1411_5373_amd as F  # noqa: E402


@pytest.mark.parametrize("band", [(0.4, 0.8), (0.1, 0.2)])
def test_heavy_ranges_are_split(band):
    """37 tiles of 448 samples and the offsets' two; ranges of 28 rows
    that read 250 to 300 rows make two blocks more than they did whole (38)."""
    nt, nd = 16384, 1024
    items = [s["work_items"] for s in F.Plan(1024, nt, nd, *band, host_only=True).steps(True)]
    tiles = (nt + nd + 447) // 448
    assert items[0] >= tiles * 40


@pytest.mark.parametrize("nf,nt,nd", [(1024, 16384, 1024), (4096, 65536, 2048), (256, 30000, 300)])
def test_even_ranges_stay(nf, nt, nd):
    """Narrow sub-bands, whose ranges read about as many rows each, keep theirs."""
    items = [s["work_items"] for s in F.Plan(nf, nt, nd, 1.2, 1.6, host_only=True).steps(True)]
    assert items == {1024: [1560, 1470, 1855], 4096: [11476, 12495, 14522], 256: [1729, 1452]}[nf]
