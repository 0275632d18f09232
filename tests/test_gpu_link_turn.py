"""Operators on link fields beyond the Infinity Cache, whose launches load the
links of their first and last tiles plainly and the others non-temporally: the
same bits as with plain loads everywhere."""
import pytest
import torch

from paper_1710_09178_amd import stag
from tests.gpu_util import log

pytestmark = pytest.mark.gpu


# 302 MB each (FP64-18, FP64-12, links and long links), and 366 MB in a number of
# tiles that is no multiple of eight, the last one ragged
@pytest.mark.parametrize("dims,links12,naik", [((32, 32, 32, 16), False, False), ((32, 32, 32, 24), True, False),
                                               ((32, 32, 32, 8), False, True), ((34, 30, 26, 24), False, False)])
def test_loads_at_the_turn_change_nothing(dims, links12, naik):
    log(f"link loads at the turn dims={dims} links12={links12} naik={naik}")
    g = torch.Generator(device="cuda").manual_seed(7)
    nx, ny, nz, nt = dims
    U = torch.randn((nt, nz, ny, nx, 4, 3, 3, 2), generator=g, device="cuda", dtype=torch.float64)
    lat = stag.Lattice(dims)
    lat.set_gauge(torch.view_as_complex(U))
    if naik:
        lat.set_naik()
    if links12:
        lat.set_link_format(stag.LINKS_F64_12)
    v, out, ref = lat.new_vec(), lat.new_vec(), lat.new_vec()
    v.copy_(torch.randn(v.shape, generator=g, device="cuda", dtype=torch.float64).to(v.dtype))
    for apply in (lambda o: lat.mdagm(o, v, 0.1), lambda o: lat.dslash(o, v, 1), lambda o: lat.dslash(o, v, 0)):
        lat.set_link_streaming(0)
        apply(ref)
        for mode in (1, 2):
            lat.set_link_streaming(mode)
            out.zero_()
            apply(out)
            assert torch.equal(out, ref)
