"""GPU: tokens with NaN logits.  Their results are unspecified, but they stay in bounds: k in
[1, K], k different expert ids below N, counts that are those of the ids (the expert GEMMs
trust them), and the other tokens' results are not touched."""
import numpy as np
import pytest
import torch

from paper_2608_04401_amd import binding as B
from paper_2608_04401_amd import synth

from helpers import RTOL_BF16, cpu, rel_err_rows, to_gpu

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _in_bounds(k, ids, N, K):
    k, ids = cpu(k), cpu(ids)
    assert k.min() >= 1 and k.max() <= K
    used = np.arange(ids.shape[1])[None, :] < k[:, None]
    assert ids[used].min() >= 0 and ids[used].max() < N
    rows = np.sort(np.where(used, ids, -1 - np.arange(ids.shape[1])[None, :]), axis=1)
    assert (np.diff(rows, axis=1) != 0).all()  # no expert twice in a token
    return used, ids


@pytest.mark.parametrize("T,d,N,K", [(5, 128, 8, 4), (300, 128, 5, 5), (4096, 64, 16, 8),
                                     (333, 128, 60, 16), (1000, 256, 64, 8),
                                     (5000, 256, 64, 8), (9000, 256, 64, 8),
                                     (9000, 256, 64, 16), (5000, 128, 60, 8), (8300, 64, 8, 4),
                                     (4200, 320, 64, 16)])
@pytest.mark.parametrize("mode", [B.MODE_ELBOW, B.MODE_TOPK])
def test_layer_with_nan_tokens(T, d, N, K, mode):
    """One in seven tokens NaN (both signs), in the one-launch router (N < 64 and N = 64), the
    split router's two routings (T = 5000 and 9000) and the one-kernel router (decode with few
    experts, and above 4096 tokens)."""
    L = synth.moe_layer(T, d, N, 64, dtype="bf16", seed=T + N)
    x, Wr, Wgu, Wd = (to_gpu(a, BF) for a in (L.x, L.W_router, L.W_gu, L.W_down))
    bad = torch.arange(T, device="cuda") % 7 == 2
    xn = x.clone().view(torch.int16)
    xn[bad, 0] = 0x7fc0
    xn[torch.arange(T, device="cuda") % 14 == 2, 0] = -64  # 0xffc0
    y, dbg = B.elb_moe_forward(xn.view(BF), Wr, Wgu, Wd, K=K, mode=mode, debug=True)
    want, ref = B.elb_moe_forward(x, Wr, Wgu, Wd, K=K, mode=mode, debug=True)
    torch.cuda.synchronize()
    used, ids = _in_bounds(dbg["k"], dbg["ids"], N, K)
    assert np.array_equal(cpu(dbg["counts"]), np.bincount(ids[used], minlength=N))
    ok = ~bad
    for name in ("logits", "k", "ids", "w"):
        assert torch.equal(dbg[name][ok], ref[name][ok])
    # the same rows in other tiles: each output within the layer's tolerance of the other
    assert rel_err_rows(cpu(y[ok]), cpu(want[ok])).max() < RTOL_BF16
