"""Device memory of the proposal network's inference: its activations for a chunk of signals, and
nothing that only training needs."""
import pytest
import torch

from paper_2007_03800_amd import api

pytestmark = pytest.mark.gpu


def test_inference_allocates_no_gradients():
    """A network too wide for the fused kernel: what the layers' activations take for 65,536 signals, with
    room for a quarter of the eight partial gradients that training keeps."""
    H, A, chunk = 2048, 256, 65536
    net = api.Proposer(8, 8, 16, 16, hidden=H)
    Y = torch.randn(64, 8, 8, device="cuda")
    api.Proposer(8, 8, 16, 16, hidden=64).logits(Y)  # torch's and the runtime's own start-up
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    out = net.logits(Y)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    # inputs, two layers' pre-activations, activations and gradients, logits and their gradient, loss parts
    batch = chunk * (2 * 64 + 2 * (4 + 2 + 2) * H + (4 + 2) * A + 8)
    partials = 8 * 4 * net.num_params
    assert used <= batch + partials // 4, (used, batch, partials)
    loss, g = net.gradient(Y, torch.zeros((64, 8), dtype=torch.int32, device="cuda"), 8)  # training still has them
    assert loss > 0 and g.shape == (net.num_params,) and out.shape == (64, A)
