"""The one-launch step (append + read, sketchssm_step) against writing the
ring slot and making the call it stands for: bitwise equal outputs, state,
sketch, map and ring, over windows of both classes with the flush in either
chunk, the single-token update, the exact baseline and rank tables; and the
tensors the kernels cannot read as they are, which take the two-call path."""
import pytest
import torch

from paper_2609_33051_amd import binding, inputs
from paper_2609_33051_amd.layer import SketchSSMLayer

pytestmark = pytest.mark.gpu

BUFFERS = ("S", "U", "cmap", "rk", "rv", "rbeta", "rla", "rf", "rpi", "rt")
CASES = [  # family, K, V, r, W, io, sketch, pivots, baseline, rank table
    ("mamba2", 128, 64, 16, 16, "bf16", "f32", 0, False, None),
    ("mamba2", 64, 64, 8, 5, "f32", "bf16", 4, False, None),
    ("mamba2", 128, 128, 32, 21, "bf16", "bf16", 4, False, None),
    ("gdn", 128, 128, 16, 16, "bf16", "bf16", 4, False, None),
    ("gdn", 64, 64, 8, 12, "f32", "f32", 0, False, [8, 0, 3]),
    ("gdn", 128, 64, 16, 20, "bf16", "f32", -1, False, None),
    ("kda", 128, 128, 16, 16, "f32", "f32", 0, False, [0, 16, 9]),
    ("kda", 128, 128, 32, 32, "bf16", "bf16", 0, False, None),
    ("kda", 64, 64, 64, 7, "bf16", "f32", 0, False, None),
    ("mamba2", 128, 64, 0, 1, "bf16", "f32", 0, True, None),
    ("gdn", 128, 128, 0, 1, "f32", "f32", 0, True, None),
    ("kda", 128, 128, 0, 1, "bf16", "f32", 0, True, None),
    ("gdn", 128, 128, 0, 6, "bf16", "f32", 0, True, None),
    ("kda", 128, 64, 0, 18, "f32", "f32", 0, True, None),
]


def _pair(fam, K, V, r, W, io, sketch, pivots, baseline, table, batch=3):
    wl = inputs.tiny(fam, batch=batch, heads=3, dk=K, dv=V, rank=max(r, 8), window=W, io=io)
    om, C = (torch.as_tensor(x) for x in inputs.omega(wl))
    S = inputs.initial_state(wl, "cuda")
    layers = [SketchSSMLayer(fam, batch, 3, K, V, r, W, io, "cuda", baseline=baseline, S=S,
                             omega=None if baseline else om, coef=None if baseline else C, sketch=sketch,
                             pivots=pivots, head_ranks=table) for _ in range(2)]
    for lay in layers:
        lay.init_sketch()
    return wl, layers


def _equal(a, b):
    for name in BUFFERS:
        x, y = getattr(a, name), getattr(b, name)
        assert (x is None) == (y is None)
        if x is not None:
            assert torch.equal(x, y), name


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c[:6])) + f"-p{c[7]}")
def test_step_is_the_append_and_the_read(case, monkeypatch):
    fam, K, V, r, W, io, sketch, pivots, baseline, table = case
    wl, (one, two) = _pair(*case)
    launched = []
    real = binding.sketchssm_step
    monkeypatch.setattr(binding, "sketchssm_step", lambda *a, **k: (launched.append(1), real(*a, **k))[1])
    steps = 2 * W + 1
    for t in range(steps):
        inp = inputs.step_inputs(wl, t, "cuda")
        a = one.step(inp).clone()
        two.write_token(inp)
        b = two.read(inp["q"]).clone()
        assert one.n == two.n
        assert torch.equal(a, b), t
    assert len(launched) == steps
    _equal(one, two)


def test_tensors_the_kernels_cannot_read_are_copied(monkeypatch):
    """A strided key, a half-precision value, a broadcast gate, a misaligned
    decay and a subclass with its own append: the same results through the slot."""
    class Own(SketchSSMLayer):
        appended = 0

        def write_token(self, inp, slot=None):
            self.appended += 1
            super().write_token(inp, slot)

    wl, (one, two) = _pair("gdn", 128, 128, 16, 8, "bf16", "f32", 0, False, None)
    monkeypatch.setattr(binding, "sketchssm_step", lambda *a, **k: pytest.fail("not laid out as the kernels read"))
    for t in range(9):
        inp = inputs.step_inputs(wl, t, "cuda")
        inp["beta"] = torch.full_like(inp["beta"], 0.5)
        plain = dict(inp)
        which = t % 4
        if which == 0:
            wide = torch.empty((3, 3, 256), dtype=torch.bfloat16, device="cuda")
            wide[..., ::2] = inp["k"]
            inp["k"] = wide[..., ::2]
        elif which == 1:
            inp["v"] = inp["v"].float()
        elif which == 2:
            inp["beta"] = torch.full((1, 1), 0.5, device="cuda").expand(3, 3)
        else:
            shifted = torch.empty(3 * 3 + 1, device="cuda")[1:].view(3, 3)
            inp["log_decay"] = shifted.copy_(inp["log_decay"])
        a = one.step(inp).clone()
        two.write_token(plain)
        assert torch.equal(a, two.read(inp["q"])), t
    _equal(one, two)
    own = Own("gdn", 3, 3, 128, 128, 16, 8, "bf16", "cuda", omega=one.omega, coef=one.coef)
    own.step(inputs.step_inputs(wl, 0, "cuda"))
    assert own.appended == 1
