"""Which wave codes a signal depends on the number of signals; its codes do not, and its early stop is
counted once.  Large signals, one wave each: workgroups of four, eight and twelve waves (up to 1,024, 2,048
signals and beyond).  Any-shape kernel: few signals spread over the workgroups, one wave's in each first."""
import pytest
import torch

from paper_2007_03800_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
def test_codes_do_not_depend_on_the_number_of_signals(dtype):
    g = torch.Generator().manual_seed(3)
    unit = lambda n, m: torch.nn.functional.normalize(torch.randn(n, m, generator=g, dtype=torch.float64), dim=1).cuda()  # noqa: E731
    D1, D2 = unit(48, 32), unit(36, 24)
    Y = torch.randn(4100, 24, 32, generator=g).to("cuda", dtype)
    Y[5::31] = 0

    def code(Y):
        pr, st = api.Problem(Y, D1, D2, 20), api.new_stats()
        api.sparse_code(pr, stats=st)
        torch.cuda.synchronize()
        return pr, st.early_stops

    whole, early = code(Y)
    assert early == len(Y[5::31]) == int((whole.supp[:, -1] < 0).sum())
    for k0, k1 in ((0, 13), (0, 1024), (1024, 2049), (2049, 4100)):
        part, early = code(Y[k0:k1])
        assert early == int((whole.supp[k0:k1, -1] < 0).sum())
        for f in ("supp", "coef", "res2"):
            assert torch.equal(getattr(whole, f)[k0:k1], getattr(part, f)), (k0, k1, f)


# four signals a wave, then one: one workgroup, a few, 256, a second wave in some, the last spread size and beyond
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("m1,m2,n1,n2,s,N,parts", [
    (9, 7, 13, 11, 6, 16400, (1, 5, 1024, 1025, 3072, 3073, 15360, 15361)),
    (8, 8, 32, 32, 8, 4100, (1, 255, 256, 257, 768, 769, 1792, 1793, 3840, 3841))])
def test_any_shape_codes_do_not_depend_on_the_number_of_signals(m1, m2, n1, n2, s, N, parts, dtype):
    g = torch.Generator().manual_seed(4)
    unit = lambda n, m: torch.nn.functional.normalize(torch.randn(n, m, generator=g, dtype=torch.float64), dim=1).cuda()  # noqa: E731
    D1, D2 = unit(n1, m1), unit(n2, m2)
    Y = torch.randn(N, m2, m1, generator=g).to("cuda", dtype)
    Y[3::29] = 0

    def code(Y):
        pr, st = api.Problem(Y, D1, D2, s), api.new_stats()
        api.sparse_code(pr, kernel=1, stats=st)
        torch.cuda.synchronize()
        return pr, st.early_stops

    whole, early = code(Y)
    assert early == len(Y[3::29]) == int((whole.supp[:, -1] < 0).sum())
    for n in parts:
        part, early = code(Y[N - n:])
        assert early == int((whole.supp[N - n:, -1] < 0).sum()), n
        for f in ("supp", "coef", "res2"):
            assert torch.equal(getattr(whole, f)[N - n:], getattr(part, f)), (n, f)
