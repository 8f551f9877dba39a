"""Packing of canonical rows: launches of many group images go four groups to a workgroup, small ones one group; units of 64 rows
are independent, so the image of all rows is the images of ranges of rows one behind the other."""
import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G4", [15, 16, 17, 18])              # 3, 4, 1 and 2 groups in the last workgroup of a unit
@pytest.mark.parametrize("O", [128, 256])
def test_many_rows_are_the_ranges(G4, O):
    rows, step = 64 * 150 - 37, 64 * 25                       # 150 units: more than 2048 images; 25: fewer; the last unit is cut
    assert 150 * G4 > 2048 >= 25 * G4
    check(rows, step, G4, O)


@pytest.mark.parametrize("G4,units", [(15, 200), (16, 200), (17, 200), (18, 200), (12, 236), (4, 720), (6, 500),      # four groups to a workgroup
                                      (1, 2900), (3, 1000), (5, 600), (9, 320)])      # one, as in the ranges
def test_many_images_are_the_ranges(G4, units):
    assert G4 * units > 2816
    check(64 * units - 37, 64 * max(1, 2000 // G4), G4, 128)


def check(rows, step, G4, O):
    print(f"[case] pack {rows} rows, {G4} INT4 groups, {O} outliers", flush=True)
    K = 128 * G4 + O
    g = torch.Generator(device="cuda").manual_seed(G4 + O)
    q4 = torch.randint(0, 256, (rows, 64 * G4), generator=g, device="cuda").to(torch.uint8)
    q8 = torch.randint(-128, 128, (rows, O), generator=g, device="cuda").to(torch.int8)
    sc = torch.rand((rows, K // 128), generator=g, device="cuda").half()
    nbytes = lambda n: atom.atom_w4a4_gemm_packed_workspace_bytes(n, 64, K, 128, O)
    pack = lambda lo, hi: atom.atom_pack_act(q4[lo:hi], q8[lo:hi], sc[lo:hi], 128,
                                             out=torch.full((nbytes(hi - lo),), 0xA5, dtype=torch.uint8, device="cuda"))
    ranges = [pack(lo, min(rows, lo + step)) for lo in range(0, rows, step)]
    assert torch.equal(pack(0, rows), torch.cat(ranges))
