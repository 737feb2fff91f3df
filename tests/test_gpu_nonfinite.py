"""Non-finite hidden states (reading R25): a token whose row holds NaN or Inf
gets NaN router scores; its selection follows the documented rule of each
mode and never exceeds what the workspace holds, and every other token of the
call is unaffected -- its mask is identical to a call without the bad
tokens and its output row finite and equal to that call's: bit for bit in
EAT mode, where the bad tokens select nothing and the experts in use are the
same, to the bf16 tolerance in the baselines, where the bad tokens' experts
join the call's and so may change the number of reduction slices the
expert kernels take (an order of additions); and the EAT accounts equal
those of a call with the bad tokens removed (snapshot semantics: tokens are
independent)."""
import numpy as np
import pytest
import torch

from paper_2609_33614_amd import _lib as L
from paper_2609_33614_amd.layer import EatLayer, to_device
from tests import parity as PT
from workload import SHAPES, HiddenStream, bf16_bits, make_accounts, make_layer_weights

pytestmark = pytest.mark.gpu

MODES = {"eat": L.EAT_MODE_EAT, "topk": L.EAT_MODE_TOPK, "topp": L.EAT_MODE_TOPP}
BAD = {3: np.nan, 10: np.inf, 11: -np.inf}


def _bf16_rows(x_bits: np.ndarray) -> torch.Tensor:
    if x_bits.dtype == np.float32:
        return torch.from_numpy(np.ascontiguousarray(x_bits)).cuda()
    return torch.from_numpy(np.ascontiguousarray(x_bits)).view(torch.bfloat16).cuda()


def _layer(shape_name, E, d, F, mode, T):
    shape = SHAPES[shape_name]
    w = make_layer_weights(shape, E=E, d=d, F=F)
    dt = L.EAT_BF16 if shape.bf16 else L.EAT_F32
    p = L.eat_params_default(mode=MODES[mode], E=E, d_model=d, d_ffn=F, top_k=shape.K, act_dtype=dt, expert_dtype=dt,
                             top_p=shape.top_p or 0.6, inv_temperature=shape.inv_temp)
    return shape, EatLayer(p, T, to_device(w))


def _run(lay, x, acc):
    if acc is not None:
        lay.load_accounts(*acc)
    mask = lay.mask_tensor(x.shape[0])
    y = lay.forward(x, mask_out=mask)
    torch.cuda.synchronize()
    return y.view(torch.int16).cpu(), PT.masks_to_list(mask), lay.accounts_host()


@pytest.mark.parametrize("mode", ["eat", "topk", "topp"])
@pytest.mark.parametrize("shape_name,E,d,F", [("finegrained", 64, 256, 256), ("qwen3", 128, 256, 256)])
def test_nonfinite_tokens_are_contained(shape_name, E, d, F, mode):
    _check_contained(shape_name, E, d, F, mode, 37)


@pytest.mark.parametrize("mode", ["eat", "topk", "topp"])
@pytest.mark.parametrize("shape_name,E,d,F,T", [
    ("finegrained", 64, 256, 256, 100),      # 128-row MFMA tiles
    ("mixtral", 4, 256, 256, 600),           # prefill tiles (300 rows per expert)
    ("tiny", 8, 128, 256, 70),               # fp32 tiles
])
def test_nonfinite_tokens_of_larger_calls(shape_name, E, d, F, T, mode):
    _check_contained(shape_name, E, d, F, mode, T)


def _check_contained(shape_name, E, d, F, mode, T):
    shape, lay = _layer(shape_name, E, d, F, mode, T)
    good = HiddenStream(shape, T, d=d, seed=5).next()                       # bf16 bits, or fp32
    bad = good.copy()
    for t, v in BAD.items():
        row = np.full(d, v, dtype=np.float32)
        bad[t] = bf16_bits(row) if shape.bf16 else row
    acc = make_accounts(E, seed=9, c_scale=0.05) if mode == "eat" else None

    yb, mb, ab = _run(lay, _bf16_rows(bad), acc)
    yg, mg, ag = _run(lay, _bf16_rows(good), acc)
    keep = [t for t in range(T) if t not in BAD]
    for t in keep:
        assert mb[t] == mg[t], t
        if mode == "eat":
            assert torch.equal(yb[t], yg[t]), t
        else:
            fb, fg = (v[t].view(torch.bfloat16 if shape.bf16 else torch.float32).float() for v in (yb, yg))
            assert torch.isfinite(fb).all(), t
            assert (fb - fg).abs().max() <= PT.TOL_Y_BF16 * fg.abs().max(), t
    K = shape.K
    for t in BAD:
        k = bin(mb[t]).count("1")
        if mode == "eat":
            assert k == 0                       # no importance beats a NaN threshold, no maximiser
            assert not yb[t].any()              # no expert: y = 0
        elif mode == "topk":
            assert mb[t] == (1 << K) - 1        # ranks collapse to 0: the K lowest indices are kept
        else:
            assert k == E                       # the running sum never reaches p: every expert
    if mode == "eat":
        # the bad tokens select nothing: the accounts equal a call without them
        _, _, a_removed = _run(lay, _bf16_rows(good[keep]), acc)
        for u, v in zip(ab, a_removed):
            np.testing.assert_array_equal(u, v)
    lay.close()


@pytest.mark.parametrize("T", [37, 100, 300])
def test_vanishing_gates(T):
    """silu(g) of g near -88 is about 1e-37, a normal number although
    1 / (1 + e^-g) is not, and counts where the up projection is large: on
    the streaming kernel, the 128-row tiles and the prefill tiles."""
    d = F = 256
    g = torch.linspace(-85.0, -88.5, F).to(torch.bfloat16)
    w1, w3, w2 = torch.zeros(1, F, d), torch.zeros(1, F, d), torch.eye(d, F)[None]
    w1[0, :, 0] = g.float()
    w3[0, :, 0] = 2.0 ** 100
    x = torch.zeros(T, d, dtype=torch.bfloat16)
    x[:, 0] = 1.0
    w = {"w_router": torch.zeros(1, d), "w1": w1.to(torch.bfloat16), "w3": w3.to(torch.bfloat16),
         "w2": w2.to(torch.bfloat16)}
    p = L.eat_params_default(mode=L.EAT_MODE_TOPK, E=1, d_model=d, d_ffn=F, top_k=1)
    lay = EatLayer(p, T, {k: v.cuda() for k, v in w.items()})
    y = lay.forward(x.cuda())
    torch.cuda.synchronize()
    ref = torch.nn.functional.silu(g.double()) * 2.0 ** 100
    # two bf16 roundings, and e^-g off by 2^-24 of its exponent 88 log2(e) and a few roundings
    assert ((y.cpu().double() - ref[None]).abs() <= (2 * 2.0 ** -8) * ref.abs()).all()
    lay.close()
