"""GPU parity of the fp32 expert GEMM (matrix instructions, 64-row tiles) and the fp32 router at
the edges of their tiles and chunks."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2608_04401_amd import binding as B
from paper_2608_04401_amd import synth

from helpers import RTOL_F32, cpu, rel_err_rows, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,m", [(16, 16), (32, 48), (80, 32), (112, 96), (144, 176)])
def test_f32_tile_edges(d, m):
    """Experts with 0, 1, 16, 17, 32, 33, 63 .. 65 and 130 rows; contractions that end in a half
    k-tile (16 of 32 columns) or are nothing else; last N-tiles of 16 to 48 columns."""
    counts = [0, 1, 16, 17, 32, 33, 63, 64, 65, 130]
    N, T = len(counts), sum(counts)
    L = synth.moe_layer(T, d, N, m, dtype="f32", seed=d + m)
    rng = np.random.default_rng(d)
    ids = rng.permutation(np.repeat(np.arange(N), counts)).astype(np.int32)[:, None]
    k = np.ones(T, np.int32)
    w = rng.uniform(0.1, 1.0, (T, 1)).astype(np.float32)
    y = B.elb_moe_experts(to_gpu(L.x), to_gpu(L.W_gu), to_gpu(L.W_down),
                          to_gpu(k, torch.int32), to_gpu(ids, torch.int32), to_gpu(w))
    torch.cuda.synchronize()
    ref = O.moe_experts(L.x, L.W_gu, L.W_down, k, ids, w.astype(np.float64))
    assert rel_err_rows(cpu(y), ref).max() < RTOL_F32


@pytest.mark.parametrize("T,d,N", [(1, 1, 2), (17, 5, 17), (16, 127, 16), (33, 130, 5),
                                   (40, 128, 64), (31, 260, 33), (5, 1024, 60)])
def test_f32_router_chunks(T, d, N):
    """One to nine chunks of 128 columns with 4- and 16-byte loads (d % 4), partial token and
    expert blocks: within the bound of an fp32 chain, d 2^-24 sum |x w|, of the exact sum."""
    rng = np.random.default_rng(d)
    x = rng.standard_normal((T, d)).astype(np.float32)
    W = rng.standard_normal((N, d)).astype(np.float32)
    got = cpu(B.elb_router_logits(to_gpu(x), to_gpu(W))).astype(np.float64)
    x64, W64 = x.astype(np.float64), W.astype(np.float64)
    assert (np.abs(got - x64 @ W64.T) <= d * 2.0 ** -24 * (np.abs(x64) @ np.abs(W64).T)).all()


def test_f32_router_unaligned_rows():
    """Rows that start off a 16-byte boundary (a view into a larger buffer) give the bits of the
    same rows aligned."""
    g = torch.Generator().manual_seed(3)
    x, W = torch.randn(20, 64, generator=g), torch.randn(18, 64, generator=g)
    buf = torch.empty(20 * 64 + 1, device="cuda")
    view = buf[1:].view(20, 64)
    view.copy_(x)
    want = B.elb_router_logits(x.cuda(), W.cuda())
    assert torch.equal(B.elb_router_logits(view, W.cuda()), want)
