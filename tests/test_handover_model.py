"""The hand-over state of the single-launch MLP, played through on the CPU: calls of different token counts, layer widths and
forms on one workspace, with the layout and the arithmetic that the kernels use (tests/handover_model.cpp)."""
import itertools
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("handover") / "model")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", os.path.join(HERE, "handover_model.cpp"), "-o", exe],
                   check=True)

    def play(sequences):
        res = subprocess.run([exe], input="".join(" ".join(s) + "\n" for s in sequences), capture_output=True, text=True,
                             check=True)
        return res.stdout.splitlines()

    return play


def _call(form, I, T, E=128, base=0):
    return f"{form}:{I}:{E}:{T}:{base}"


def _check(model, sequences):
    for seq, verdict in zip(sequences, model(sequences)):
        assert verdict == "ok", f"{' '.join(seq)}: {verdict}"


@pytest.mark.parametrize("I", [64, 512, 1024, 2048, 4096, 8192])
def test_token_counts_on_one_workspace(model, I):
    """Every pair of (form, tokens) in turn, and all orders of three of the smallest: all workgroups of each launch see one epoch, and no other launch of the call did."""
    forms = [("words", T) for T in (1, 2, 3, 4)] + [("slots", T) for T in (1, 2, 3, 4, 5, 8, 13, 16, 32, 64)] + [("plain", 65)]
    pairs = [[_call(*x) for x in ((a, I, s), (b, I, t), (a, I, s), (a, I, s))] for (a, s), (b, t) in itertools.permutations(forms, 2)]
    triples = [[_call(a, I, t) for a, t in order] * 2 for order in itertools.permutations(forms[:4] + [("slots", 5)], 3)]
    _check(model, pairs + triples)


@pytest.mark.parametrize("form", ["words", "slots"])
def test_layers_of_different_width_on_one_workspace(model, form):
    """The layers of a model, or of two, share one workspace (the library's own array is one for all shapes)."""
    widths = (64, 256, 1024, 2048, 4096, 4864, 5632, 8192, 11008, 14336)
    seqs = [[_call(f, i, t, e) for f, i, t, e in ((form, a, s, 64), (form, b, t, 2048), (form, a, s, 64), (form, a, s, 2048))]
            for a, b in itertools.permutations(widths, 2) for s, t in ((1, 1), (1, 2), (4, 1))]
    _check(model, seqs)


def test_other_uses_of_the_memory(model):
    """Between two launches the memory is written from its first byte on, as the MLP on E5M2 weights does, or in any pieces of
    512 bytes, as an allocator hands it round."""
    again = [_call("words", 1024, 1), _call("slots", 1024, 5)]
    _check(model, [[_call("words", I, T), _call("low", J, S), _call("words", I, T), _call("words", I, T)]
                   for I in (1024, 4096, 8192) for T in (1, 2, 4) for J in (64, 512, 2048, 8192) for S in (1, 5)])
    _check(model, [again + [f"pieces:{first}:0:{n}"] + again * 2 for first in range(18) for n in (1, 2, 3, 17)])


def test_workspaces_that_begin_elsewhere_in_the_same_memory(model):
    """Nothing holds two calls in a row to one place: a second workspace lies over a part of the first one."""
    at = lambda base, T: _call("words", 1024, T, base=base)
    _check(model, [[at(a, 1), at(b, 2), at(a, 1), at(a, 3), at(b, 2), at(a, 1)]
                   for a in (0, 256, 4096) for b in range(0, 16384, 256) if a != b])
