"""Row pitch of the ghosted state: whole 128-byte lines, unless that alone would
take the state past the 4 GiB that the fused kernels address."""
import pytest

from paper_2306_14011_amd import fv, inputs


@pytest.mark.parametrize("n,pitch", [
    ((1, 1), 16), ((12, 5), 16), ((13, 5), 32), ((2048, 2048), 2064), ((97, 61, 45), 112), ((256, 256, 256), 272),
    ((11572, 11580), 11584),          # 16-double rows: 4.294050e9 bytes, below 2^32
    ((11572, 11586), 11576),          # 16-double rows would take 4.296e9 bytes
    ((11572, 11600), 11576),          # above 2^32 either way
    ((470, 470, 470), 480), ((476, 476, 472), 480),
    ((481, 472, 470), 488),           # 16-double rows: 496 * 476 * 474 * 40 bytes > 2^32 > 488 * 476 * 474 * 40
], ids=str)
def test_row_pitch(n, pitch):
    g = inputs.grid2d(*n) if len(n) == 2 else inputs.grid3d(*n)
    sx, sy, sz, sv = fv.fv_query(fv.make_desc(g))[0]
    assert (sx, sy) == (1, pitch)
    assert sz == sy * (n[1] + 4) and sv == sz * (n[2] + 4 if len(n) == 3 else 1)
