"""GPU parity of the mid-sized expert GEMM kernel (64- and 128-row tiles) at the edges of its
tiles, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2608_04401_amd import binding as B
from paper_2608_04401_amd import synth

from helpers import RTOL_BF16, cpu, rel_err_rows, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,m", [(64, 64), (192, 64), (320, 192), (128, 128), (64, 576)])
def test_mid_tile_edges(d, m):
    """Experts with 0, 1, 63 .. 65, 127 .. 129, 192, 193 and 256 rows: both tile forms, one to
    three tiles sharing their weights, one to nine k-tiles (started at every N-tile's own one),
    a last N-tile of 64 of 128 columns (d = 64, 192, 320)."""
    counts = [0, 1, 63, 64, 65, 127, 128, 129, 192, 193, 256]
    N, T = len(counts), sum(counts)
    L = synth.moe_layer(T, d, N, m, dtype="bf16", seed=d + m)
    rng = np.random.default_rng(d)
    ids = rng.permutation(np.repeat(np.arange(N), counts)).astype(np.int32)[:, None]
    k = np.ones(T, np.int32)
    w = rng.uniform(0.1, 1.0, (T, 1)).astype(np.float32)
    x, Wgu, Wd = (to_gpu(a, torch.bfloat16) for a in (L.x, L.W_gu, L.W_down))
    y = B.elb_moe_experts(x, Wgu, Wd, to_gpu(k, torch.int32), to_gpu(ids, torch.int32),
                          to_gpu(w))
    torch.cuda.synchronize()
    ref = O.moe_experts(L.x, L.W_gu, L.W_down, k, ids, w.astype(np.float64))
    # bf16 storage of H and of the expert output: two roundings of 2^-9 relative
    assert rel_err_rows(cpu(y), ref).max() < RTOL_BF16


@pytest.mark.parametrize("d", [192, 512])
def test_large_kernel_short_tiles(d):
    """The 256-row kernel's tiles of at most 64 and 128 rows: alone (experts of 1, 40, 65 and 128
    rows) and behind full tiles (256 + 33 .. 129 rows), a last N-tile of 192 of 256 columns
    (d = 192), an odd number of k-tiles (d = 192: three), started in the middle in the odd
    N-tiles of the lone ones."""
    counts = [1, 40, 65, 128, 289, 320, 321, 384, 385, 700, 900]
    N, T, m = len(counts), sum(counts), 1024
    assert T // N >= 112 and (T + 128 * N) // 256 * (m // 128) > 128  # the 256-row kernel
    L = synth.moe_layer(T, d, N, m, dtype="bf16", seed=d)
    rng = np.random.default_rng(d)
    ids = rng.permutation(np.repeat(np.arange(N), counts)).astype(np.int32)[:, None]
    k = np.ones(T, np.int32)
    w = rng.uniform(0.1, 1.0, (T, 1)).astype(np.float32)
    x, Wgu, Wd = (to_gpu(a, torch.bfloat16) for a in (L.x, L.W_gu, L.W_down))
    y = B.elb_moe_experts(x, Wgu, Wd, to_gpu(k, torch.int32), to_gpu(ids, torch.int32),
                          to_gpu(w))
    torch.cuda.synchronize()
    ref = O.moe_experts(L.x, L.W_gu, L.W_down, k, ids, w.astype(np.float64))
    assert rel_err_rows(cpu(y), ref).max() < RTOL_BF16


@pytest.mark.parametrize("d,m,crowd", [(128, 1024, 0), (192, 1024, 0), (320, 1024, 0),
                                       (576, 384, 9000), (320, 128, 31000)])
def test_large_kernel_lone_full_tiles(d, m, crowd):
    """The 256-row kernel's full tiles of experts that have one (129 to 256 rows), whose odd
    N-tiles start in the middle of the contraction: two, three and five k-tiles in gate/up (d =
    128, 192, 320), two and six in down (m = 128, 384, beside an expert of `crowd` rows that makes
    the problem large enough), a last N-tile of 64 columns (d = 320, 576)."""
    counts = [129, 130, 191, 192, 255, 256, 200, 257, 512] + [140 + 8 * i for i in range(11)]
    if crowd:
        counts[-1] = crowd
    N, T = len(counts), sum(counts)
    assert T // N >= 112 and (T + 128 * N) // 256 * (m // 128) > 128  # the 256-row kernel
    L = synth.moe_layer(T, d, N, m, dtype="bf16", seed=d + m)
    rng = np.random.default_rng(d)
    ids = rng.permutation(np.repeat(np.arange(N), counts)).astype(np.int32)[:, None]
    k = np.ones(T, np.int32)
    w = rng.uniform(0.1, 1.0, (T, 1)).astype(np.float32)
    x, Wgu, Wd = (to_gpu(a, torch.bfloat16) for a in (L.x, L.W_gu, L.W_down))
    y = B.elb_moe_experts(x, Wgu, Wd, to_gpu(k, torch.int32), to_gpu(ids, torch.int32),
                          to_gpu(w))
    torch.cuda.synchronize()
    others = ids[:, 0] < N - 1 if crowd else np.ones(T, bool)
    tok = np.sort(np.concatenate([np.nonzero(others)[0], np.nonzero(~others)[0][:512]]))
    ref = O.moe_experts(L.x, L.W_gu, L.W_down, k[tok], ids[tok], w[tok].astype(np.float64),
                        tokens=tok)
    assert rel_err_rows(cpu(y)[tok], ref).max() < RTOL_BF16
