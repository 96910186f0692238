"""The pair pass's split count, as the working memory of the allocation-free
energy call shows it: every split holds points (chunks of 256; an empty one would
write and add rows of zeros)."""
import pytest

CHUNK, TARGET = 256, 8192


def up(x, to=256):
    return (x + to - 1) // to * to


def splits(n, n_atom):
    """Splits and padded points of a grid of n points."""
    from paper_2208_14639_amd import vv10
    npad = up(n)
    # packed points (FP64, FP32), 15 fields, 6 integrals, atom indices, reduction
    # scratch, flags; then six rows of partials per split where there are several
    fixed = sum(map(up, (32 * npad, 32 * npad, 16 * npad, 16 * npad, 15 * 8 * npad, 6 * 8 * npad,
                         4 * npad, 8 * max(npad // 256 + 2, 195), 4 * (n_atom + 2))))
    rows = vv10.vv10_noalloc_bytes(n, n_atom) - fixed
    assert rows >= 0 and rows % (48 * npad) == 0, (n, rows)
    return max(1, rows // (48 * npad)), npad


@pytest.mark.parametrize("n", [1, 255, 257, 1500, 4200, 4352, 6000, 9000, 12000, 27000, 36864, 51000,
                               101949, 120000, 225000])
def test_no_split_is_empty(n):
    s, npad = splits(n, 6)
    per = -(-(npad // CHUNK) // s)                 # chunks of a split
    assert 1 <= s <= 16
    assert (s - 1) * per < npad // CHUNK <= s * per
    # the target of workgroups is met as far as 16 splits of whole chunks can
    # (within the scratch of the allocation-free call, which fits all of these)
    want = min(16, -(-TARGET // (npad // 64)), npad // CHUNK)
    assert s == -(-(npad // CHUNK) // -(-(npad // CHUNK) // max(1, want))) or 268 * npad + 48 * want * npad > (63 << 20)


@pytest.mark.parametrize("n,n_atom", [(129537, 300000), (180993, 300000), (128001, 500000),
                                      (124161, 1000000), (180993, 1000000), (72193, 5000000),
                                      (175361, 5000000)])
def test_splits_leave_room_for_the_atoms(n, n_atom):
    """A grid that fits the allocation-free call's scratch without partials keeps
    fitting, however many (empty) atoms its flags count."""
    from paper_2208_14639_amd import vv10
    assert 0 < vv10.vv10_noalloc_bytes(n, n_atom) <= vv10.VV10_NOALLOC_SCRATCH_BYTES
    splits(n, n_atom)
