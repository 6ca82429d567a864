"""The per-step tensor helpers as native functions: the arguments, results and errors of the Python ones they replace."""
import inspect
import os
import pickle
import subprocess
import sys

import pytest
import torch

from paper_2503_06545_amd import binding as qc

qc._use_native_helpers()   # binding may have been imported before torch
REPLACED = sorted(qc._python_helpers)


def outcome(f, *args, **kwargs):
    try:
        return f(*args, **kwargs)
    except Exception as e:   # the type and the text are what is compared
        return type(e), str(e)


def test_all_are_replaced_under_their_signatures():
    assert REPLACED == sorted(qc._PER_STEP)
    for n in REPLACED:
        native, python = inspect.signature(getattr(qc, n)), inspect.signature(qc._python_helpers[n])
        assert [(p.name, p.default, p.kind) for p in native.parameters.values()] == [
            (p.name, p.default, p.kind) for p in python.parameters.values()]


@pytest.mark.parametrize("before", ["", "import torch; ", "from paper_2503_06545_amd.binding import qlinear_t; import torch; "])
def test_a_pickled_helper_works_in_another_process(before):
    """What was pickled here, or by a program that took the helpers from the module before it imported torch, is called
    in a process that has imported nothing yet."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    for n in REPLACED:
        f = getattr(qc, n)
        assert f.__doc__ == (inspect.getdoc(qc._python_helpers[n]) or None) and pickle.loads(pickle.dumps(f)) is f
        assert pickle.loads(pickle.dumps(qc._python_helpers[n])) is qc._python_helpers[n]
    code = f"""
import sys, pickle
sys.path.insert(0, {root!r})
{before}
for f in pickle.loads({pickle.dumps([getattr(qc, n) for n in REPLACED] + [qc._python_helpers[n] for n in REPLACED])!r}):
    try:
        f(1, 2, 3)
    except Exception as e:
        assert type(e) is AttributeError, repr(e)
"""
    subprocess.run([sys.executable, "-c", code], check=True, timeout=100)


@pytest.fixture
def handed_on():
    """The calls that the native helpers hand on to the Python ones, by name."""
    from paper_2503_06545_amd import _qc_torch
    seen = []

    def recorded(n):
        def helper(*args, **kwargs):
            seen.append(n)
            return qc._python_helpers[n](*args, **kwargs)
        return helper

    _qc_torch.setup(qc._entries, qc._check, tuple(recorded(n) for n in qc._PER_STEP))
    yield seen
    _qc_torch.setup(qc._entries, qc._check, tuple(qc._python_helpers[n] for n in qc._PER_STEP))


class NoPointer(torch.Tensor):
    """A subclass: the Python helper's business."""


def test_what_is_refused_is_refused_alike(handed_on):
    x, w = torch.zeros(2, 16, dtype=torch.bfloat16), torch.zeros(512, dtype=torch.uint8)
    pw, ws, y, f = qc.PackedWeight(w, torch.zeros(3), 3, 16, 8), torch.zeros(4096, dtype=torch.uint8), torch.zeros(2, 3), torch.zeros(4, 4)
    calls = [("qlinear_t", (), {}), ("qlinear_t", (x,), {}), ("qlinear_t", (x, pw), {}), ("qlinear_t", (x, pw, None, "no"), {}),
             ("qlinear_t", (x, pw), {"workspace": ws, "Y": y}), ("qlinear_t", (x, pw), {"X": x}), ("qlinear_t", (x, pw), {"nothing": 1}),
             ("qlinear_t", (x, None), {"workspace": ws, "Y": y}), ("qlinear_t", (x, pw, None, "none", "f32", ws, y, 8, 0, 1), {}),
             ("qlinear_t", (x.as_subclass(NoPointer), pw), {"workspace": ws, "Y": y}), ("qlinear_t", (1, pw), {"workspace": ws, "Y": y}),
             ("qlinear_asym_t", (x, pw, None), {"workspace": ws, "Y": y}), ("qlinear_tensor_t", (x, pw), {"workspace": ws, "Y": y, "act_bits": 8.0}),
             ("latent_delta_t", (f, f), {"workspace": ws, "out3": y}), ("latent_delta_t", (f, None), {"workspace": ws, "out3": y}),
             ("layer_similarity_t", (f, f[:2]), {"workspace": ws, "out4": y}), ("frame_gradient_norm_t", (f,), {"workspace": ws, "out2": y}),
             ("cumulative_variation_t", (f, [f, f]), {"workspace": ws, "out": y}), ("cumulative_variation_t", (f, f), {"workspace": ws, "out": y})]
    for name, args, kwargs in calls:
        want = outcome(qc._python_helpers[name], *args, **kwargs)
        handed_on.clear()
        assert isinstance(want, tuple) and outcome(getattr(qc, name), *args, **kwargs) == want, (name, args, kwargs)
        assert handed_on == [name]


@pytest.mark.gpu
def test_results_and_device_errors_are_those_of_the_python_helpers(handed_on):
    """Ordinary calls are the native helpers' own, also where the library refuses them; those that leave out the workspace and the
    output or bring tensors of another type, order or container go to the Python helpers."""
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(40, 256, generator=g, device="cuda").bfloat16()
    pw, prw = (qc.pack_weight_t(torch.randn(72, 256, generator=g, device="cuda"), 8, rot) for rot in (0, 64))
    bias, sums = torch.randn(72, generator=g, device="cuda"), qc.weight_row_sums_t(pw)
    a, b = (torch.randn(3, 1000, generator=g, device="cuda") for _ in range(2))

    def space(make):
        return {"workspace": make(40, 256, 72), "Y": torch.empty(40, 72, dtype=torch.bfloat16, device="cuda")}

    def small(key, count):
        return {"workspace": torch.empty(1 << 16, dtype=torch.uint8, device="cuda"), key: torch.empty(count, device="cuda")}

    little = {"workspace": torch.empty(16, dtype=torch.uint8, device="cuda"), "Y": torch.empty(40, 72, device="cuda")}
    own = [("qlinear_t", (x, pw), lambda: dict(space(qc.qlinear_workspace_t), bias=bias, epi="gelu_tanh", act_bits=6)),
           ("qlinear_t", (x, prw), lambda: dict(space(qc.qlinear_workspace_t), rot_block=64)),
           ("qlinear_t", (x, pw, None, "none", "bf16", *space(qc.qlinear_workspace_t).values()), dict),
           ("qlinear_asym_t", (x, pw, sums), lambda: dict(space(qc.qlinear_asym_workspace_t), bias=bias)),
           ("qlinear_tensor_t", (x, pw), lambda: dict(space(qc.qlinear_tensor_workspace_t), epi="gelu_erf")),
           ("latent_delta_t", (a, b), lambda: small("out3", 3)), ("layer_similarity_t", (a, b), lambda: small("out4", 4)),
           ("layer_similarity_t", (x, x), lambda: small("out4", 4)), ("frame_gradient_norm_t", (a,), lambda: small("out2", 2)),
           ("cumulative_variation_t", (a, [b, a, b]), lambda: small("out", 4)), ("qlinear_t", (x, pw), lambda: little),
           ("qlinear_t", (x, pw), lambda: dict(space(qc.qlinear_workspace_t), act_bits=5))]
    others = [("qlinear_t", (x, pw, bias), dict), ("latent_delta_t", (a, b), dict), ("qlinear_t", (x.double(), pw), lambda: space(qc.qlinear_workspace_t)),
              ("qlinear_t", (x.t(), pw), lambda: space(qc.qlinear_workspace_t)), ("latent_delta_t", (a, b.t()), lambda: small("out3", 3)),
              ("cumulative_variation_t", (a, [b] * 9), lambda: small("out", 10)), ("cumulative_variation_t", (a, (b, a)), lambda: small("out", 3))]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            for i, (name, args, options) in enumerate(own + others):
                given = options()
                want = outcome(qc._python_helpers[name], *args, **options())
                if torch.is_tensor(want):
                    want = want.clone()   # of the call that was given its output by position
                handed_on.clear()
                got = outcome(getattr(qc, name), *args, **given)
                assert handed_on == ([] if i < len(own) else [name]), (name, given)
                if isinstance(want, tuple):
                    assert got == want, (name, got, want)
                    continue
                stream.synchronize()
                assert torch.equal(got, want), name
                assert not given or any(got is v for v in given.values())
