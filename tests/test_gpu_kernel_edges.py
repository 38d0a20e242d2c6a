"""The single-token update's tile map and the flush's masked slots at the sizes
where they can go wrong, against the recurrence in 64 bits (plain torch)."""
import pytest
import torch

from paper_2609_33051_amd import binding, inputs
from paper_2609_33051_amd.layer import SketchSSMLayer

pytestmark = pytest.mark.gpu

# fp32 sums over at most 128 channels and 16 tokens: a few units in the last
# place of the result (2^-24 = 6e-8 each), as the parity bar for fp32 storage
REL = 1e-5


def _step64(kind, S, tok):
    """X <- X Diag(alpha), erase, write; o = X q (X [B][H][V][K], 64 bits)."""
    q, k, v, beta, ld = (tok[x].double() for x in ("q", "k", "v", "beta", "log_decay"))
    S = S * torch.exp(ld if ld.dim() == 3 else ld[..., None])[:, :, None, :]
    w = beta[..., None] * (v - (S * k[:, :, None, :]).sum(-1) if kind != "mamba2" else v)
    S = S + w[..., None] * k[:, :, None, :]
    return S, (S * q[:, :, None, :]).sum(-1)


def _rel(a, b):
    return float((a.double() - b).norm() / b.norm())


@pytest.mark.parametrize("kind", ["mamba2", "gdn", "kda"])
@pytest.mark.parametrize("K,V", [(64, 64), (128, 64), (128, 128)])
@pytest.mark.parametrize("B,H", [(1, 1), (1, 7), (2, 4), (3, 3), (5, 7)])
def test_single_token_update_of_any_item_count(kind, K, V, B, H):
    """One wave per 16-value tile, eight items dealt to the XCDs at a time: item
    counts below eight, a multiple of eight and with a remainder."""
    for io in ("f32", "bf16"):
        wl = inputs.tiny(kind, batch=B, heads=H, dk=K, dv=V, rank=8, window=1, io=io)
        S = inputs.initial_state(wl, "cuda")
        lay = SketchSSMLayer(kind, B, H, K, V, 0, 1, io, "cuda", baseline=True, S=S)
        X = S.double()
        for t in range(3):
            tok = inputs.step_inputs(wl, t, "cuda")
            X, o = _step64(kind, X, tok)
            assert _rel(lay.step(tok), o) < REL, (io, t)
            assert _rel(lay.rv[:, :, 0], tok["v"].double()) == 0.0 and _rel(lay.rk[:, :, 0], tok["k"].double()) == 0.0
        assert _rel(lay.state(), X) < REL, io


@pytest.mark.parametrize("kind", ["mamba2", "gdn", "kda"])
@pytest.mark.parametrize("K,V", [(64, 64), (128, 128)])
@pytest.mark.parametrize("W", [2, 3, 4, 5, 13, 15, 16, 17, 19, 31])
def test_flush_of_any_window(kind, K, V, W):
    """Slots past the window are masked by zeros in LDS, not by branches: every
    remainder of a slot group and of a 16-slot chunk."""
    wl = inputs.tiny(kind, batch=2, heads=3, dk=K, dv=V, rank=16, window=W, io="bf16")
    S = inputs.initial_state(wl, "cuda")
    om, C = (torch.as_tensor(x) for x in inputs.omega(wl))
    lay = SketchSSMLayer(kind, 2, 3, K, V, 16, W, "bf16", "cuda", S=S, omega=om, coef=C)
    lay.init_sketch()
    for name in ("rk", "rv"):  # slots not yet written must not show in the reads (the flush uses every slot)
        getattr(lay, name).fill_(float("nan"))
    X = S.double()
    for t in range(W):
        tok = inputs.step_inputs(wl, t, "cuda")
        X, o = _step64(kind, X, tok)
        got = lay.step(tok)
    assert _rel(got, o) < REL
    assert _rel(lay.state(), X) < REL
    assert _rel(lay.sketch_matrix(), torch.stack([X[:, h] @ om[h].cuda().double() for h in range(3)], 1)) < REL


@pytest.mark.parametrize("kind", ["mamba2", "gdn", "kda"])
@pytest.mark.parametrize("K,V", [(64, 64), (128, 64), (128, 128)])
@pytest.mark.parametrize("W,m", [(16, 1), (16, 5), (16, 13), (16, 16), (32, 15), (32, 16), (32, 17), (32, 18), (32, 27)])
@pytest.mark.parametrize("pivots", [0, 4])
def test_early_flush_ignores_unused_slots(kind, K, V, W, m, pivots):
    """A window flushed after m tokens, with NaN in everything the flush has no
    business with: ring slots m and on, and the rows of T^{-1} from slot m - 1
    on, their diagonals and what lies above."""
    wl = inputs.tiny(kind, batch=3, heads=3, dk=K, dv=V, rank=16, window=W, io="bf16")
    S = inputs.initial_state(wl, "cuda")
    om, C = (torch.as_tensor(x) for x in inputs.omega(wl))
    lay = SketchSSMLayer(kind, 3, 3, K, V, 16, W, "bf16", "cuda", S=S, omega=om, coef=C, pivots=pivots)
    lay.init_sketch()
    X = S.double()
    for t in range(m):
        tok = inputs.step_inputs(wl, t, "cuda")
        X, o = _step64(kind, X, tok)
        if t < m - 1:
            lay.step(tok)
    lay.write_token(tok, m - 1)
    for name in ("rk", "rv", "rbeta", "rla"):
        getattr(lay, name)[:, :, m:] = float("nan")
    if lay.rt is not None:
        s, j = torch.meshgrid(torch.arange(W), torch.arange(W), indexing="ij")
        unused = ((s >= m - 1) | (j >= s)).cuda()
        lay.rt.permute(0, 3, 1, 2)[unused] = float("nan")  # [slot][column][H][B]
    got = torch.empty_like(lay.o)
    binding.sketchssm_update(lay.cfg, lay.S, lay.omega, lay.ring, m - 1, tok["q"], lay.U, got, lay.stream(), cmap=lay.cmap)
    assert _rel(got, o) < REL
    assert _rel(lay.state(), X) < REL
    assert _rel(lay.sketch_matrix(), torch.stack([X[:, h] @ om[h].cuda().double() for h in range(3)], 1)) < REL
    if pivots:
        assert bool(torch.isfinite(lay.cmap).all())


def test_kda_flush_that_forgets_a_channel():
    """A log decay of minus infinity on the window's last token (alpha = 0)
    clears those channels' past and leaves the other channels alone."""
    W = 6
    wl = inputs.tiny("kda", batch=2, heads=2, dk=128, dv=128, rank=16, window=W, io="f32")
    S = inputs.initial_state(wl, "cuda")
    om, C = (torch.as_tensor(x) for x in inputs.omega(wl))
    lay = SketchSSMLayer("kda", 2, 2, 128, 128, 16, W, "f32", "cuda", S=S, omega=om, coef=C)
    lay.init_sketch()
    X = S.double()
    for t in range(W):
        tok = inputs.step_inputs(wl, t, "cuda")
        if t == W - 1:
            tok["log_decay"][..., ::5] = float("-inf")
        X, o = _step64("kda", X, tok)
        got = lay.step(tok)
    assert bool(torch.isfinite(lay.state()).all())
    assert _rel(got, o) < REL and _rel(lay.state(), X) < REL


@pytest.mark.parametrize("kind", ["mamba2", "gdn"])
@pytest.mark.parametrize("W", [1, 6, 16, 17, 21])
def test_flush_that_forgets_everything(kind, W):
    """A scalar log decay of minus infinity on the window's last token: the state
    is that token's write alone."""
    wl = inputs.tiny(kind, batch=2, heads=2, dk=128, dv=128, rank=16, window=W, io="f32")
    S = inputs.initial_state(wl, "cuda")
    lay = SketchSSMLayer(kind, 2, 2, 128, 128, 0, W, "f32", "cuda", baseline=True, S=S)
    X = S.double()
    for t in range(W):
        tok = inputs.step_inputs(wl, t, "cuda")
        if t == W - 1:
            tok["log_decay"].fill_(float("-inf"))
        X, o = _step64(kind, X, tok)
        got = lay.step(tok)
    assert _rel(got, o) < REL and _rel(lay.state(), X) < REL


@pytest.mark.parametrize("kind", ["gdn", "kda"])
@pytest.mark.parametrize("K,V", [(64, 64), (128, 128)])
@pytest.mark.parametrize("W", [2, 6, 16, 17, 32])
def test_flush_with_an_infinite_value(kind, K, V, W):
    """An infinite value on the last token reaches its own value channel as it
    does in the recurrence (infinities with the sign of the key), with no NaN,
    and no other channel; earlier in the window, no other channel."""
    for slot in {W - 1, W // 2}:
        wl = inputs.tiny(kind, batch=2, heads=2, dk=K, dv=V, rank=16, window=W, io="f32")
        S = inputs.initial_state(wl, "cuda")
        lay = SketchSSMLayer(kind, 2, 2, K, V, 0, W, "f32", "cuda", baseline=True, S=S)
        X = S.double()
        for t in range(W):
            tok = inputs.step_inputs(wl, t, "cuda")
            if t == slot:
                tok["v"][..., 5] = float("inf")
            X, o = _step64(kind, X, tok)
            got = lay.step(tok)
        state = lay.state()
        rest = [i for i in range(V) if i != 5]
        assert _rel(state[:, :, rest], X[:, :, rest]) < REL and _rel(got[..., rest], o[..., rest]) < REL
        if slot == W - 1:
            assert torch.equal(state[:, :, 5].double(), X[:, :, 5])
