"""Aggregations on a graph whose rows without entries lie before, between and
after the others, at widths that leave lanes of the last 64 columns idle:
every row is written, with the values of a full-width call."""
import numpy as np
import pytest
import torch

import paper_2010_07565_amd as bg
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    bg.load()
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def graph(dev):
    """A third of the nodes have rows (of an R-MAT graph), the rest none."""
    g = workloads.rmat_graph(20_001, 300_000, 6)
    n = 3 * g.n + 500
    deg = np.zeros(n, dtype=np.int64)
    deg[250:250 + 3 * g.n:3] = np.diff(g.rowptr)
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    colidx = (3 * g.colidx.astype(np.int64) + 250).astype(np.int32)
    return n, torch.from_numpy(rowptr).to(dev), torch.from_numpy(colidx).to(dev)


@pytest.mark.parametrize("K", [64, 65])
@pytest.mark.parametrize("d,full", [(65, 128), (127, 128), (129, 256), (255, 256), (3, 4),
                                    (40, 64)])
def test_every_row_is_written(dev, graph, K, d, full):
    """A row of the 8-bit layout does not depend on the width within 65-128
    or 129-256 columns, so the first d columns of the full-width call are
    the narrower call's, bit for bit."""
    n, rowptr, colidx = graph
    gen = torch.Generator(device=dev).manual_seed(K + d)
    h = torch.randn((n, K), device=dev, generator=gen)
    wbits, alpha = bg.pack_weights(torch.randn((full, K), device=dev, generator=gen))
    bias = torch.randn(full, device=dev, generator=gen)
    F = torch.empty((n, bg.words(K)), dtype=torch.int64, device=dev)
    g = torch.empty(n, device=dev)
    bg.bigcn_binarize_pack(h, F, g, None, None, rowptr, "mean")
    C8 = torch.empty((n, bg.q8_row(full)), dtype=torch.int8, device=dev)
    C16 = torch.empty((n, bg.q8_row(full)), dtype=torch.float16, device=dev)
    bg.bigcn_bgemm_q8(F, wbits, K, C8, C16, g)
    cself = torch.empty((n, full), dtype=torch.float16, device=dev)
    bg.bigcn_bgemm(F, wbits, K, cself)
    ws = torch.empty(bg.spmm_workspace_bytes(n, colidx.numel(), full), dtype=torch.uint8,
                     device=dev)
    outs = []
    for w in (full, d):
        a, b = alpha[:w].contiguous(), bias[:w].contiguous()
        o = torch.full((n, w), float("nan"), device=dev)
        bg.bigcn_spmm_csr_q8(rowptr, colidx, g, C8, C16, K, a, o, ws, b, "mean", d=w)
        s = torch.full((n, w), float("nan"), device=dev)
        bg.bigcn_spmm_csr_sage_q8(rowptr, colidx, g, C8, C16, K, a, cself, a, s, ws, b, d=w)
        outs.append((o[:, :d], s[:, :d]))
    torch.cuda.synchronize()
    for x, y in zip(*outs):
        assert bool(torch.isfinite(y).all())
        assert torch.equal(x, y)
