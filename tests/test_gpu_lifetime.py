"""GPU: a problem's workspace may be freed after hom_destroy, also when its
set-up (which is queued without a wait) has not run yet: the release waits for
the problem's stream.  Other work queued before the set-up keeps it pending."""
import pytest

import homgen

pytestmark = pytest.mark.gpu

CASES = [("2d", (23, 13), "mixed"), ("2d_fp64", (41, 41), "fp64"), ("3d", (5, 13, 13), "mixed")]


def _cell(N):
    return homgen.sphere_cell(seed=2, n=3, anisotropic=True) if len(N) == 3 else homgen.random_squares_cell(2)[0]


@pytest.mark.parametrize("after", ["setup", "update", "net_input"])
@pytest.mark.parametrize("name,N,prec", CASES, ids=[c[0] for c in CASES])
def test_release_waits_for_queued_work(name, N, prec, after):
    import torch
    import paper_1404_3614_amd as H
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    cell = _cell(N)
    Ah, Bh, nc = H.coef_from_cell(cell, N)
    st = torch.cuda.Stream()
    big = torch.ones((8192, 8192), device="cuda")
    big @ big                                # library and code objects loaded
    H.Problem(len(N), N, cell.Y, Ah, Bh, precision=prec, ncoef=nc, stream=st)
    torch.cuda.synchronize()

    def busy():                              # tens of milliseconds on the problem's stream alone
        with torch.cuda.stream(st):
            out = torch.empty_like(big)
            for _ in range(6):
                torch.mm(big, big, out=out)
        return out

    keep = busy()
    pb = H.Problem(len(N), N, cell.Y, Ah, Bh, precision=prec, ncoef=nc, stream=st)
    if after != "setup":                     # only the later call is pending
        torch.cuda.synchronize()
        keep = busy()
        if after == "update":
            pb.stream.wait_stream(torch.cuda.current_stream())
            H._lib.check(H._lib.load().hom_update_coefficients(pb.h, Ah.data_ptr(), Bh.data_ptr()), "update")
        else:
            out = torch.empty((2,) + pb.M, dtype=torch.float32, device="cuda")
            H._lib.check(H._lib.load().hom_net_input(pb.h, out.data_ptr()), "net_input")
    assert not st.query(), "the stream is meant to be busy here"
    n = pb.ws.numel()
    del pb
    assert st.query(), "released with work still queued"
    t = torch.full((n,), 7, dtype=torch.uint8, device="cuda")   # takes the workspace's memory
    torch.cuda.synchronize()
    assert bool((t == 7).all())
    del keep
