"""Large signals, one wave each: workgroups of four, eight and twelve waves by the number of signals (up to
1,024, 2,048 and beyond) give every signal the same codes, and count its early stop once."""
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
