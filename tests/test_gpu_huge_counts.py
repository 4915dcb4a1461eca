"""More planes, or images, than a launch of one workgroup (one wave) for each could count threads for: 2^32 threads is where
the runtime cuts a grid off without an error.  The first and the last of them are looked at."""
import pytest

pytestmark = pytest.mark.gpu


def test_scan_of_more_planes_than_one_launch_holds():
    import torch
    import paper_2512_07884_amd as G
    from paper_2512_07884_amd import binding
    C, H, W = (1 << 24) + 1000, 9, 11
    x = torch.ones((1, C, H, W), dtype=torch.bfloat16, device="cuda")
    x[0, -3:] = 2.0
    one = torch.ones((1, 1, 1, 1, 1), dtype=torch.bfloat16, device="cuda").expand(1, 1, C, H, W).contiguous()
    w = torch.zeros((1, 1, 1, 3, H, W), dtype=torch.bfloat16, device="cuda")         # no propagation: y = 4 x
    y = torch.full_like(x, float("nan"))
    G.gspn_scan_fwd(x, w, one, one, y, None, G=1, flags=binding.GSPN_FLAG_SHARED_PARAMS)
    torch.cuda.synchronize()
    assert bool((y[0, :1000] == 4).all()) and bool((y[0, -2000:-3] == 4).all()) and bool((y[0, -3:] == 8).all())


def test_projection_of_more_images_than_one_launch_holds():
    import torch
    import paper_2512_07884_amd as G
    B = (1 << 26) + 1000                                                              # one wave per image
    x = torch.ones((B, 8, 1, 9), dtype=torch.bfloat16, device="cuda")
    x[-3:] = 2.0
    P = torch.ones((1, 8), dtype=torch.bfloat16, device="cuda")
    out = torch.full((B, 1, 1, 9), float("nan"), dtype=torch.bfloat16, device="cuda")
    G.gspn_proxy_project(x, P, out)
    torch.cuda.synchronize()
    assert bool((out[:1000] == 8).all()) and bool((out[-2000:-3] == 8).all()) and bool((out[-3:] == 16).all())
