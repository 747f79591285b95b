"""The launch grid of the fp32 expert GEMMs (csrc/tilegrid.h): enough blocks, whole rows on the same
XCD order, and no dimension whose threads reach 2^32, where a launch wraps around."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_04401_amd", "csrc")

PROG = r'''
#include <cstdio>
#include "tilegrid.h"
int main() {
    long long n;
    while (scanf("%lld", &n) == 1) {
        const elb::TileGrid g = elb::tile_grid(n);
        printf("%lld %u %u\n", n, g.x, g.y);
    }
}
'''


def test_tile_grid():
    sizes = [1, 7, 8, 9, 1000, 2 ** 23 - 1, 2 ** 23, 2 ** 23 + 1, 2 ** 24 - 1, 2 ** 24,
             2 ** 24 + 1, 131135 * 128, 2 ** 26 + 3, 2 ** 30]
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "t.cpp"), os.path.join(d, "t")
        open(src, "w").write(PROG)
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, src, "-o", exe])
        out = subprocess.run([exe], input="\n".join(map(str, sizes)), text=True, check=True,
                             stdout=subprocess.PIPE).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert [r[0] for r in rows] == sizes
    for n, x, y in rows:
        assert x % 8 == 0 and x * 256 < 2 ** 32 and 1 <= y <= 65535
        assert n <= x * y < n + x + 8
        assert x == 2 ** 23 if y > 1 else n <= 2 ** 23  # the row of the kernel's block number


@pytest.mark.gpu
def test_f32_gate_up_of_more_than_2_24_blocks():
    """fp32, 2^17 tokens with 64 slots each (one used), d = 16, m = 4096: 131135 x 128 tiles at
    most, 16.8 M blocks of 256 threads.  Every 64-bit result of 512 tokens spread over the
    batch; the scratch is 138 GB, of which the used rows (2 GB) are touched."""
    import torch

    from paper_2608_04401_amd import binding as B
    T, d, N, m, K = 1 << 17, 16, 64, 4096, 64
    need = B.elb_moe_workspace_bytes(T, d, N, m, K, B.ELB_F32)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < need + (8 << 30):
        pytest.skip("needs %.0f GB of free GPU memory" % (need / 1e9))
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.randn((T, d), generator=g, device="cuda")
    Wgu = torch.randn((N, 2 * m, d), generator=g, device="cuda") * 0.1
    Wd = torch.randn((N, d, m), generator=g, device="cuda") * 0.1
    ids = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
    ids[:, 0] = torch.randint(0, N, (T,), generator=g, device="cuda", dtype=torch.int32)
    w = torch.zeros((T, K), device="cuda")
    w[:, 0] = 1.0
    k = torch.ones(T, dtype=torch.int32, device="cuda")
    y = torch.empty_like(x)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    rc = B.lib().elb_moe_experts(x.data_ptr(), Wgu.data_ptr(), Wd.data_ptr(), k.data_ptr(),
                                 ids.data_ptr(), w.data_ptr(), None, T, d, N, m, K, B.ELB_F32,
                                 y.data_ptr(), ws.data_ptr(), ws.numel(), B._stream())
    assert rc == 0
    torch.cuda.synchronize()
    del ws
    torch.cuda.empty_cache()
    tok = torch.arange(0, T, T // 512, device="cuda") + 77
    e, xs = ids[tok, 0].long().cpu(), x[tok].double().cpu()
    Wg, Wd64 = Wgu.double().cpu(), Wd.double().cpu()
    for i in range(len(tok)):
        h = Wg[e[i]] @ xs[i]
        ref = Wd64[e[i]] @ (torch.nn.functional.silu(h[:m]) * h[m:])
        # fp32 sums of 16 and 4096 products: 1e-4, the layer's fp32 tolerance
        assert (y[tok[i]].double().cpu() - ref).norm() < 1e-4 * ref.norm()
