"""Host checks of the default forward schedule (no GPU): which calls take block
passes, which keep their own form, and that no accepted length is refused."""
import pytest

torch = pytest.importorskip("torch")

import paper_1411_5373_amd as F  # noqa: E402

KINDS = F.binding.STEP_KINDS


def _plan(nf, nt, nd, **kw):
    return F.Plan(nf, nt, nd, 1.2, 1.6, host_only=True, **kw)


def test_default_schedule_takes_block_passes():
    for nf, passes in ((64, 1), (128, 2), (1024, 2), (4096, 2), (8192, 3)):
        s = _plan(nf, 5000, 64).steps()
        assert len(s) == passes and s[0]["kind"] == KINDS[6] and all(x["kind"] == KINDS[5] for x in s[1:])
        assert all(0 < x["lds_bytes"] <= 65536 for x in s)
        assert s[0]["level_first"] == 0 and s[-1]["level_last"] == nf.bit_length() - 1
    # a channel count that is no power of two needs no padded copy
    assert [x["kind"] for x in _plan(1000, 5000, 64).steps()] == [KINDS[6], KINDS[5]]
    # long Option-1 chains: the initialisation on its own
    assert _plan(32, 5000, 2000).steps()[0]["kind"] == KINDS[0]


@pytest.mark.parametrize("kw", [dict(first_kernel=2), dict(first_kernel=3), dict(first_levels=3), dict(later_levels=2),
                                dict(gather_rows=4), dict(gather_threads=512), dict(tile=256), dict(lds_kib=64),
                                dict(first_rows=2), dict(first_threads=512), dict(stream_tiles=2), dict(later_kernel=1)])
def test_explicit_fields_keep_their_form(kw):
    a, b = _plan(1000, 5000, 300).steps(), _plan(1000, 5000, 300, **kw).steps()
    assert b[0]["kind"] == KINDS[9] and a[0]["kind"] == KINDS[6]  # the padded copy is the other forms'


def test_search_keeps_a_register_pass():
    s = _plan(1024, 5000, 300, search_rows=2).steps()
    assert s[-1]["lds_bytes"] == 0 and s[-1]["level_first"] == 8 and s[-1]["level_last"] == 10


def test_lengths_past_the_block_tiles_are_still_accepted():
    ok = 65535 * 224
    assert _plan(64, ok, 64, gather_vecs=2).steps()[0]["lds_bytes"] > 0
    # more tiles than the grid's y dimension holds: the other forms' wider ones
    s = _plan(64, 2 * ok, 64, gather_vecs=2).steps()
    assert s[0]["kind"] == KINDS[2]
    assert _plan(4, 5000, 30).steps()[0]["kind"] == KINDS[2]  # fewer than three iterations


def test_adjoint_block_passes():
    for nf, passes in ((16, 1), (64, 2), (1024, 3), (4096, 3), (8192, 4)):
        s = _plan(nf, 5000, min(nf, 64)).steps(True)
        assert len(s) == passes and all(x["kind"] == KINDS[8] and x["lds_bytes"] > 0 for x in s)
        assert s[0]["level_last"] == nf.bit_length() - 1 and s[-1]["level_first"] == 0
    # long chains keep the transposed initialisation on its own
    assert _plan(32, 5000, 2000).steps(True)[-1]["kind"] == KINDS[4]
    for kw in (dict(adjoint_levels=2), dict(adjoint_last_levels=2), dict(gather_rows=8), dict(gather_vecs=2),
               dict(adjoint_rows=4), dict(adjoint_threads=512), dict(adjoint_tile_major=1)):
        assert all(x["lds_bytes"] == 0 for x in _plan(1024, 5000, 64, **kw).steps(True))
    # past the block tiles, or with shifts that need too many more of them: the register gathers
    assert all(x["lds_bytes"] == 0 for x in _plan(64, 65535 * 500, 64).steps(True))
    assert all(x["lds_bytes"] == 0 for x in _plan(64, 5000, 64, d_min=1 << 30).steps(True))


def test_adjoint_windows():
    """Windows of 512 samples (more than 40 KB of LDS) once they fill the GPU."""
    for nf, nt, nd, wide in ((256, 70001, 300, True), (2048, 20011, 1500, True), (1024, 8192, 1024, False),
                             (128, 131072, 64, False)):
        assert (_plan(nf, nt, nd).steps(True)[0]["lds_bytes"] > 40000) == wide
