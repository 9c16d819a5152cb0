"""The path's validation and vorticity in one kernel against the two separate
calls, bit for bit, on grids at the edges of its tiles (64 x 16 vectors): one
vector, fewer than three, a vector or two past a tile, several tiles; frames
of noise, so that outliers lie next to each other and across tiles."""
import pytest
import torch

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP device")]


@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 3), (63, 15), (64, 16), (65, 17), (66, 18), (67, 19), (130, 33), (2, 50),
                                   (129, 3)])
def test_run_equals_separate_validation_and_vorticity(nx, ny):
    from paper_2504_17987_amd import api
    W, H, n = 8 * nx, 8 * ny, 3
    gen = torch.Generator(device="cuda").manual_seed(nx * 1000 + ny)
    A = torch.randint(0, 256, (n, H, W), generator=gen, device="cuda", dtype=torch.uint8)
    B = torch.roll(A, (1, 2), (1, 2))
    noisy = torch.rand((n, H, W), generator=gen, device="cuda") < 0.6
    B = torch.where(noisy, torch.randint(0, 256, (n, H, W), generator=gen, device="cuda", dtype=torch.uint8), B)
    B[1, : H // 2, : W // 2] = 7   # flat windows
    P = api.Plan(W, H, max_batch=n, levels=1)
    out = P.run(A, B)
    disp, _, flags = P.correct(A, B, out["pred"])
    P.validate(disp, flags)
    omega = P.vorticity(disp)
    assert torch.equal(out["flags"], flags)
    assert torch.equal(out["disp"].view(torch.int32), disp.view(torch.int32))
    assert torch.equal(out["omega"].view(torch.int32), omega.view(torch.int32))
    if nx > 8 and ny > 8:
        assert int((flags & 8).count_nonzero()) > 0 or int(flags.count_nonzero()) > 0


def test_replacements_on_both_sides_of_tile_borders():
    """The same comparison on a field with replaced vectors in every row and
    column next to a border of the kernel's tiles (64 x 16 vectors; the last
    ones moved back to end with the grid), and next to vectors of FLAT
    windows."""
    from paper_2504_17987_amd import api
    nx, ny, n = 130, 33, 6
    W, H = 8 * nx, 8 * ny
    gen = torch.Generator(device="cuda").manual_seed(77)
    A = torch.randint(0, 256, (n, H, W), generator=gen, device="cuda", dtype=torch.uint8)
    noisy = torch.rand((n, H, W), generator=gen, device="cuda") < 0.6
    B = torch.where(noisy, torch.randint(0, 256, (n, H, W), generator=gen, device="cuda", dtype=torch.uint8),
                    torch.roll(A, (1, 2), (1, 2)))
    B[1, : H // 2, : W // 2] = 7
    P = api.Plan(W, H, max_batch=n, levels=1)
    out = P.run(A, B)
    disp, _, flags = P.correct(A, B, out["pred"])
    raw = disp.clone()
    P.validate(disp, flags)
    omega = P.vorticity(disp)
    replaced = (flags & 16) != 0
    assert torch.equal(replaced, (raw != disp).any(1) & replaced)   # (a replacement is another value)
    for x in (63, 64, 65, 66, 127, 128):
        assert replaced[:, :, x].any(), x
    for y in (15, 16, 17, 31, 32):
        assert replaced[:, y, :].any(), y
    assert (flags[1] & 1).any()
    assert torch.equal(out["flags"], flags)
    assert torch.equal(out["disp"].view(torch.int32), disp.view(torch.int32))
    assert torch.equal(out["omega"].view(torch.int32), omega.view(torch.int32))
