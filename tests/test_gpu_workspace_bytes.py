"""gf_space_cache_info reports what the workspaces hold: the dense coarse inverses stay with their plan."""
import pytest

from paper_2605_24882_amd import inputs

pytestmark = pytest.mark.gpu

g = pytest.importorskip("paper_2605_24882_amd.gfield")
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available()
    return g.Context(0)


def test_workspace_bytes_are_what_workspaces_hold(ctx):
    # one-level space: 41 dense inverses of 488 unknowns are 78 MB, a workspace of 41 or 82 columns 10 to 20 MB.  The
    # second call has the plan of the first and a workspace of its own
    sp = g.Space(ctx, g.Geometry(ctx, False), 2, 3, mg_levels=1)
    z = torch.from_numpy(inputs.noise_vectors([0, 1], sp.noise_length)).cuda()
    b = sp.white_noise(z)
    held = []
    for n in (1, 2):
        u = sp.sample(3.0, 0.6, b[:n].contiguous(), k_minus=20, k_plus=20, rtol=1e-8)[0]
        torch.cuda.synchronize()
        held.append((torch.cuda.mem_get_info()[0], sp.cache_info()))
    (free0, (p0, pb0, w0, wb0)), (free1, (p1, pb1, w1, wb1)) = held
    assert p1 == p0 and pb1 == pb0 and w1 > w0
    # blocks of the call itself and the allocator's granularity come on top: less than half the inverses
    assert free0 - free1 <= wb1 - wb0 + (30 << 20), ((free0 - free1) >> 20, (wb1 - wb0) >> 20)
