"""GPU: tensors that start off a 16-byte boundary (contiguous views into larger buffers).  The
kernels that copy with 16-byte LDS copies have a form with ordinary loads for them, or leave
them to another kernel: the same arithmetic gives the bits of the aligned call; a layer that
the large-tile GEMM would take runs the mid-sized one, within the layer's tolerance."""
import pytest
import torch

from paper_2608_04401_amd import binding as B
from paper_2608_04401_amd import synth

from helpers import RTOL_BF16, cpu, rel_err_rows, to_gpu

pytestmark = pytest.mark.gpu


def _shifted(t, elements):
    buf = torch.empty(t.numel() + elements, dtype=t.dtype, device=t.device)
    view = buf[elements:].view(t.shape)
    view.copy_(t)
    assert view.data_ptr() % 16 == elements * t.element_size() % 16
    return view


# decode (tasks by slot and by expert), mid-sized with the one-launch and the one-kernel router,
# above 4096 tokens, the large-tile kernel's sizes, fp32
@pytest.mark.parametrize("dtype,T,d,N,m,K", [
    ("bf16", 1, 256, 64, 64, 8), ("bf16", 40, 320, 16, 192, 4), ("bf16", 300, 192, 16, 128, 4),
    ("bf16", 1000, 256, 64, 64, 8), ("bf16", 4100, 256, 64, 64, 2), ("bf16", 2000, 192, 8, 1024, 2),
    ("f32", 100, 48, 8, 80, 3), ("f32", 300, 64, 5, 48, 2)])
@pytest.mark.parametrize("which", [(1, 1, 1, 1), (1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 3, 0),
                                   (0, 0, 0, 7)])
def test_unaligned_tensors(dtype, T, d, N, m, K, which):
    """which: the elements that x, W_router, W_gate_up and W_down are shifted by."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    L = synth.moe_layer(T, d, N, m, dtype=dtype, seed=T + d)
    args = [to_gpu(a, dt) for a in (L.x, L.W_router, L.W_gu, L.W_down)]
    want, ref = B.elb_moe_forward(*args, K=K, debug=True)
    y, dbg = B.elb_moe_forward(*(_shifted(a, n) if n else a for a, n in zip(args, which)), K=K,
                               debug=True)
    torch.cuda.synchronize()
    for name in ("logits", "k", "ids", "w", "counts"):
        assert torch.equal(dbg[name], ref[name])
    if T < 2000 or T > 4000:
        assert torch.equal(y, want)
    else:
        assert rel_err_rows(cpu(y), cpu(want)).max() < RTOL_BF16


@pytest.mark.parametrize("T,d,N,K", [(50, 256, 64, 8), (300, 96, 20, 12)])
def test_unaligned_router_route(T, d, N, K):
    L = synth.moe_layer(T, d, N, 64, dtype="bf16", seed=T)
    x, Wr = to_gpu(L.x, torch.bfloat16), to_gpu(L.W_router, torch.bfloat16)
    want = B.elb_router_route(x, Wr, K=K, with_logits=True)
    for a, b in ((_shifted(x, 1), Wr), (x, _shifted(Wr, 5))):
        got = B.elb_router_route(a, b, K=K, with_logits=True)
        torch.cuda.synchronize()
        assert all(torch.equal(p, q) for p, q in zip(got, want))
