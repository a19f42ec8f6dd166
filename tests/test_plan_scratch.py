"""Scratch of a best-hit call at the library's own tile height (host side, no GPU): lower tiles, which a
short plan takes to fill the chip, must not push a genome pair past the fixed scratch of
``pdp_bh_noalloc`` that it fits with the usual 64-row tiles."""
import ctypes as C

import pytest

import paper_2510_23679_amd as pdp
from paper_2510_23679_amd import binding as B


def _fake(n, residues, k, base):
    arena, _ = pdp.dict_size(n, residues, k)
    d = B.pdp_dict()
    B.check(pdp.lib().pdp_dict_bind(base, arena, n, residues, k, 0, 0, C.byref(d)), "pdp_dict_bind")
    return d


def _ws(a, b, tile_rows):
    p, n = pdp.params(tile_rows=tile_rows), C.c_uint64(0)
    B.check(pdp.lib().pdp_bh_ws_size(C.byref(a), C.byref(b), C.byref(p), C.byref(n)), "pdp_bh_ws_size")
    return n.value


@pytest.mark.parametrize("per", [100, 300, 512, 1500, 4000])
@pytest.mark.parametrize("nq", [1, 200, 3000, 10000, 30000])
def test_default_tiles_fit_the_fixed_scratch_where_64_rows_do(nq, per):
    for nt in (1, 1000, 10000, 30000):
        a, b = _fake(nq, nq * per, 6, 256), _fake(nt, nt * per, 6, 1 << 40)
        if _ws(a, b, 64) <= pdp.PDP_NOALLOC_SCRATCH_BYTES:
            assert _ws(a, b, 0) <= pdp.PDP_NOALLOC_SCRATCH_BYTES, (nq, nt, per)
