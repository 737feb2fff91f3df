"""The 128- and 256-row MFMA tiles of medium calls (more than 64 tokens, too
few rows per expert for the prefill tiles) against the oracle: one token over
a tile's rows and one under, a last weight tile that ends inside the matrix
(widths that are odd multiples of 64), the shortest reduction the ring takes
(192), sliced down projections, an always-on expert, and bit equality between
the packed and the row-major weights."""
import numpy as np
import pytest
import torch

from paper_2609_33614_amd import _lib as L
from paper_2609_33614_amd.layer import EatLayer, PplSignal, pack_weights, to_device
from tests import test_gpu_parity as P
from workload import make_accounts

pytestmark = pytest.mark.gpu

CASES = {
    # 128-row tiles: d = 192 (3 chunks, 64 rows past the second weight tile), F = 320
    "short": dict(shape="mixtral", d=192, F=320, E=8, Fs=0),
    # 32 feature tiles x 8 experts: 256-row tiles from ~100 rows per expert
    "tall": dict(shape="mixtral", d=256, F=2048, E=8, Fs=0),
    # few rows over many experts, an always-on expert of its own tiles
    "many": dict(shape="shared", d=320, F=192, E=60, Fs=448),
    # EAT's 8 experts make 64 items: the streaming kernel's 128-token tiles up to 96
    # tokens, with gate/up partials in the down projection's slices
    "few": dict(shape="finegrained", d=1024, F=512, E=64, Fs=0),
}


@pytest.mark.parametrize("case,T,mode", [
    ("short", 65, "topk"), ("short", 128, "eat"), ("short", 129, "eat"), ("short", 513, "topk"),
    ("tall", 384, "topk"), ("tall", 520, "topp"), ("tall", 900, "eat"), ("tall", 70, "eat"),
    ("many", 65, "topp"), ("many", 257, "eat"), ("many", 300, "topk"),
    ("few", 65, "eat"), ("few", 96, "eat"), ("few", 97, "eat"), ("few", 96, "topk"),
])
def test_mid_tiles(case, T, mode):
    c = CASES[case]
    shape, w, lay, prm = P._layer(c, mode, max_tokens=T)
    x = P._x_host(shape, T, c["d"], seed=T)
    acc = make_accounts(c["E"], seed=T, c_scale=0.05)
    P._forward_check(f"mid {case} {mode} T={T}", lay, shape, x, w, prm, acc=acc)

    wd = to_device(w)
    p = lay.params
    outs = []
    for layout in (L.EAT_LAYOUT_ROWS, L.EAT_LAYOUT_PACKED):
        q = type(p).from_buffer_copy(p)
        q.weight_layout = layout
        lq = EatLayer(q, T, wd if layout == L.EAT_LAYOUT_ROWS else pack_weights(wd))
        lq.load_accounts(*acc)
        y = lq.forward(P._x_dev(x))
        torch.cuda.synchronize()
        outs.append((y.view(torch.int16).cpu().numpy(), *lq.accounts_host()))
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("S,d,V", [(1, 192, 64), (16, 256, 960), (128, 192, 320), (129, 512, 1088), (383, 256, 448),
                                   (3, 128, 64)])
def test_head_tiles(S, d, V):
    """The LM head of the perplexity signal on the same tiles (d = 128: on the
    streaming kernel), against float64.  An fp32 sum of d products of bf16
    values is off by at most d 2^-24 sum |h w|, and a logsumexp by no more than
    its logits plus a few fp32 roundings of its value."""
    g = torch.Generator().manual_seed(S + d + V)
    head = (torch.randn(V, d, generator=g) * d ** -0.5).to(torch.bfloat16)
    h = torch.randn(S, d, generator=g).to(torch.bfloat16)
    target = torch.randint(0, V, (S,), generator=g).to(torch.int32)
    sig = PplSignal(S, head.cuda())
    sig.reset()
    sig.step(h.cuda(), target.cuda())
    torch.cuda.synchronize()
    z = h.double() @ head.double().T
    nll = torch.logsumexp(z, 1) - z.gather(1, target.long()[:, None])[:, 0]
    bound = 2 * d * 2.0 ** -24 * (h.double().abs() @ head.double().abs().T).max() + 16 * 2.0 ** -24 * (1 + nll.abs().max())
    assert (sig.nll.cpu().double() - nll).abs().max() <= bound


@pytest.mark.parametrize("S,d,V", [(1, 192, 64), (16, 256, 960), (128, 192, 320), (129, 512, 1088), (383, 256, 448),
                                   (384, 256, 512), (3, 128, 192), (40, 256, 33024), (64, 192, 32832)])
def test_every_head_column_counts_once(S, d, V):
    """Hidden rows along one head row each, c: its logit, 15, carries the
    sequence's logsumexp, so a lost column moves the NLL by several units and a
    repeated one by log 2 (all columns of small heads; of large ones the first and
    last tiles).  The bound is that of test_head_tiles, per sequence."""
    g = torch.Generator().manual_seed(S + d + V)
    head = (torch.randn(V, d, generator=g) * d ** -0.5).to(torch.bfloat16)
    cols = torch.arange(V) if V <= 1100 else torch.cat([torch.arange(130), torch.arange(V - 330, V)])
    sig = PplSignal(S, head.cuda())
    for i in range(0, len(cols), S):
        c = cols[torch.arange(i, i + S) % len(cols)]
        h = (15.0 * head[c].float() / head[c].float().square().sum(1, keepdim=True)).to(torch.bfloat16)
        target = (c + V // 2) % V
        sig.reset()
        sig.step(h.cuda(), target.to(torch.int32).cuda())
        torch.cuda.synchronize()
        z = h.double() @ head.double().T
        nll = torch.logsumexp(z, 1) - z.gather(1, target[:, None])[:, 0]
        bound = 2 * d * 2.0 ** -24 * (h.double().abs() @ head.double().abs().T).max(1).values + 16 * 2.0 ** -24 * (1 + nll)
        assert bound.max() < 0.05
        assert ((sig.nll.cpu().double() - nll).abs() <= bound).all(), (i, S, d, V)
