"""Routing of small routers in one launch (up to 16 experts and 16 KB): around
the 16-token groups, with one and 16 experts, one to eight k-steps a slice (odd
counts too), and at the largest router it takes and the first it leaves to
the two launches."""
import pytest
import torch

import oracle as O
from tests import test_gpu_parity as P
from workload import make_accounts, make_trend

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,E,d", [("tiny", 1, 64), ("tiny", 16, 192), ("tiny", 8, 512), ("mixtral", 16, 256),
                                       ("mixtral", 5, 448), ("mixtral", 8, 512), ("mixtral", 8, 576)])
@pytest.mark.parametrize("T,mode", [(1, "eat"), (16, "topk"), (17, "eat"), (500, "topp"), (1023, "eat"), (1024, "topk")])
def test_small_router(shape, E, d, T, mode):
    c = dict(shape=shape, d=d, F=64, E=E, Fs=0)
    s, w, lay, prm = P._layer(c, mode, K=min(2, E), max_tokens=T)
    x = P._x_host(s, T, d, seed=T + d)
    acc = make_accounts(E, seed=T, c_scale=0.05)
    trend = make_trend(T, seed=T)
    lay.load_accounts(*acc)
    mask, k, gate, prob = lay.route(P._x_dev(x), torch.from_numpy(trend).cuda())
    torch.cuda.synchronize()
    P._check_routing(f"route small E={E} d={d} {mode} T={T}", O.route(x, w["w_router"], acc, trend, prm), prm, mask,
                     gate, prob, k)
