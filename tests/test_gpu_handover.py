"""The single-launch MLP (one token tile): its in-kernel hand-over of H under graph replay, on a garbage
workspace, at the full size of the 1B-shaped layer with changing activations, and its failure handling
forced from the host (producers withhold the publication, consumers poll a few times and give up - every
kernel exits normally)."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2507_03117_amd import synth
from tests.helpers import check_close, mask_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch

    assert torch.cuda.is_available()
    from paper_2507_03117_amd import api as _api

    _api.lib()
    return _api


def _layer(api, seed, E, I, b, sparsity):
    rng = np.random.default_rng(seed)
    ws_ = [synth.gauss_bf16(rng, s, 0.05) for s in ((I, E), (I, E), (E, I))]
    ms_ = [synth.uniform_mask(rng, r // b, c // b, sparsity) for r, c in ((I, E), (I, E), (E, I))]
    ms_[2][1, :] = 0  # an empty block row of the down projection: nothing to wait for, zeros
    dev = [api.bsr_pack(to_dev(w), b, mask=mask_dev(m)) for w, m in zip(ws_, ms_)]
    ref = [orc.pack(w, b, m) for w, m in zip(ws_, ms_)]
    return rng, dev, ref, ms_


@pytest.mark.parametrize("b,T", [(64, 1), (64, 3), (64, 16), (64, 32), (64, 50), (128, 1), (128, 2), (128, 5), (128, 16), (128, 30)])
def test_single_launch_form_replays_from_a_graph(api, b, T):
    """One token tile: the call is recorded as ONE kernel and every replay - with new activations, with eager
    calls on the same workspace between the replays - hands over its own H."""
    import torch

    E, I = 4 * b, 6 * b
    rng, dev, ref, _ = _layer(api, 8100 + b + T, E, I, b, 0.5)
    ws = torch.full((max(api.mlp_workspace_bytes(*dev, T), 256),), 0x5A, dtype=torch.uint8, device="cuda:0")  # garbage
    xs = to_dev(synth.gauss_bf16(rng, (T, E), 1.0))
    y = torch.empty((T, E), dtype=torch.float32, device="cuda:0")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        api.sparse_mlp(*dev, xs, out=y, ws=ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.sparse_mlp(*dev, xs, out=y, ws=ws)
        api.sparse_mlp(*dev, xs, out=y, ws=ws)  # two launches per replay: consecutive epochs inside one graph
    for rep in range(4):
        x = synth.gauss_bf16(rng, (T, E), 1.0)
        xs.copy_(to_dev(x))
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check_close(y.cpu().numpy().T, orc.mlp(*ref, x), f"replay {rep} b={b} T={T}")
        if rep % 2 == 0:  # an eager call in between, on the same workspace
            x2 = synth.gauss_bf16(rng, (T, E), 1.0)
            y2 = api.sparse_mlp(*dev, to_dev(x2), ws=ws)
            torch.cuda.synchronize()
            check_close(y2.cpu().numpy().T, orc.mlp(*ref, x2), f"eager between replays {rep}")
    assert api.sparse_mlp_status(dev[0], T, ws) == 0


def test_single_launch_form_at_the_1b_shape_with_changing_activations(api):
    """Full-size reuse: the 1B-shaped layer, one workspace, activations changing from call to call and the token
    count moving inside the tile: no call may see H lines or slots of an earlier one."""
    import torch

    wl = synth.WORKLOADS["llama1b_b64_s90"]
    inp = synth.make_mlp(wl)
    dev = [api.bsr_pack(to_dev(l.W), wl.b, mask=mask_dev(l.mask)) for l in (inp.gate, inp.up, inp.down)]
    ref = [orc.pack(l.W, wl.b, l.mask) for l in (inp.gate, inp.up, inp.down)]
    rng = np.random.default_rng(8200)
    Tmax = 64
    ws = torch.full((api.mlp_workspace_bytes(*dev, Tmax),), 0xC3, dtype=torch.uint8, device="cuda:0")
    for rep, T in enumerate((32, 1, 17, 64, 4, 32, 47, 16, 2)):
        x = synth.gauss_bf16(rng, (T, wl.hidden), 1.0)
        # the workspace layout depends on T: give each T the prefix it asks for, as a caller with one big buffer would
        y = api.sparse_mlp(*dev, to_dev(x), ws=ws[: api.mlp_workspace_bytes(*dev, T)],
                           out=torch.full((T, wl.hidden), float("nan"), device="cuda:0"))
        torch.cuda.synchronize()
        check_close(y.cpu().numpy().T, orc.mlp(*ref, x), f"1B single launch call {rep} T={T}")
        assert api.sparse_mlp_status(dev[0], T, ws[: api.mlp_workspace_bytes(*dev, T)]) == 0


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
def test_tagged_words(api, b, T, out_dtype):
    """A few tokens: H travels as tagged words where the workspace has room for them, else through slots.  Both forms on a
    garbage workspace, with rows of the down projection of 0 to 23 blocks (a wave takes four, two or one at a time), gated and
    two-matrix; activations change from call to call on one workspace; the two forms agree up to the order of the sums."""
    import torch

    E, I = 8 * b, 24 * b
    rng = np.random.default_rng(8250 + b + T)
    shapes = ((I, E), (I, E), (E, I))
    ws_ = [synth.gauss_bf16(rng, s, 0.05) for s in shapes]
    ms_ = [synth.uniform_mask(rng, r // b, c // b, 0.5) for r, c in shapes]
    for br, count in enumerate((0, 1, 4, 5, 16, 17, 8, 23)):
        ms_[2][br] = 0
        ms_[2][br, rng.choice(I // b, size=count, replace=False)] = 1
    dev = [api.bsr_pack(to_dev(w), b, mask=mask_dev(m)) for w, m in zip(ws_, ms_)]
    ref = [orc.pack(w, b, m) for w, m in zip(ws_, ms_)]
    dt = torch.float32 if out_dtype == "f32" else torch.bfloat16
    tol = 0.0 if out_dtype == "f32" else 2.0 ** -7
    whole = api.mlp_workspace_bytes(*dev, T)
    xs = [synth.gauss_bf16(rng, (T, E), 1.0) for _ in range(3)]
    words = {}  # results of the first form, by call
    for size in (whole, whole - T * I * 8) if T <= 4 else (whole,):
        ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device="cuda:0")
        for rep, x in enumerate(xs):
            out = torch.full((T, E), float("nan"), dtype=dt, device="cuda:0")
            y = api.sparse_mlp(*dev, to_dev(x), ws=ws, out=out).float()
            want = orc.mlp(*ref, x)
            z = api.sparse_mlp2(dev[0], dev[2], to_dev(x), ws=ws, out=torch.empty_like(out)).float()
            want2 = orc.mlp2(ref[0], ref[2], x)
            torch.cuda.synchronize()
            for got, exp in ((y, want), (z, want2)):
                got = got.cpu().numpy().T
                if tol == 0.0:
                    check_close(got, exp, f"tagged b={b} T={T} ws={size} call {rep}")
                else:  # one rounding to bf16 on top of the sums
                    assert (np.abs(got - exp) <= np.abs(exp) * tol + 1e-2 * np.sqrt((exp ** 2).mean())).all()
                assert not got[:b].any()  # an empty block row
            for first, got in zip(words.setdefault(rep, (y, z)), (y, z)):
                # the same H; fp32 sums of at most 8 blocks of a wave and four waves, in whatever order, and one rounding of them
                slack = 64 * 2.0 ** -24 * float(first.abs().max()) + tol * first.abs()
                assert ((got - first).abs() <= slack).all(), f"words and slots differ, b={b} T={T} call {rep}"
        assert api.sparse_mlp_status(dev[0], T, ws) == 0


@pytest.mark.parametrize("b,I", [(64, 512), (64, 2048), (64, 4096), (128, 1024)])
def test_token_counts_and_widths_change_on_one_workspace(api, b, I):
    """A decoding program whose batch changes from call to call, and two layers of different width, on one workspace and on
    the library's own array: eager calls of both MLP forms, and graphs captured at one and two tokens replayed in turn
    between them, with new activations each time.  Every wait ends normally."""
    import torch

    E = 4 * b
    rng, dev, ref, _ = _layer(api, 8400 + b + I, E, I, b, 0.6)
    _, dev2, ref2, _ = _layer(api, 8500 + b + I, E, I + 6 * b, b, 0.6)
    size = max(api.mlp_workspace_bytes(*d, T) for d in (dev, dev2) for T in (1, 2, 3, 4, 5, 8))
    ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device="cuda:0")
    graphs = {}
    for T in (1, 2):
        xs, y = torch.zeros((T, E), dtype=torch.bfloat16, device="cuda:0"), torch.empty((T, E), device="cuda:0")
        torch.cuda.synchronize()
        graphs[T] = (torch.cuda.CUDAGraph(), xs, y)
        with torch.cuda.graph(graphs[T][0]):
            api.sparse_mlp(*dev, xs, out=y, ws=ws)

    def replay(T, what):
        graph, xs, y = graphs[T]
        x = synth.gauss_bf16(rng, (T, E), 1.0)
        xs.copy_(to_dev(x))
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        check_close(y.cpu().numpy().T, orc.mlp(*ref, x), f"{what}, replay T={T}")

    for n, T in enumerate((1, 2, 1, 4, 3, 5, 2, 8, 1)):
        for layer, (d, r) in enumerate(((dev, ref), (dev2, ref2))):
            what = f"b={b} I={I} call {n} T={T} layer {layer}"
            x = synth.gauss_bf16(rng, (T, E), 1.0)
            want = orc.mlp(*r, x)
            y = api.sparse_mlp(*d, to_dev(x), ws=ws)
            y_static = api.sparse_mlp_static(*d, to_dev(x), torch.full_like(y, float("nan")))
            z = api.sparse_mlp2(d[0], d[2], to_dev(x), ws=ws)
            torch.cuda.synchronize()
            check_close(y.cpu().numpy().T, want, what)
            check_close(y_static.cpu().numpy().T, want, what + " static")
            check_close(z.cpu().numpy().T, orc.mlp2(r[0], r[2], x), what + " two-matrix")
        replay(2 if n % 2 else 1, what)
        replay(1 if n % 2 else 2, what)
    for T in (1, 2, 3, 4, 5, 8):
        assert api.sparse_mlp_status(dev[0], T, ws) == 0
        assert api.sparse_mlp_status(dev[0], T, None) == 0


def test_workspaces_that_the_allocator_hands_round(api):
    """Calls without a workspace of the caller's get what the allocator has: memory that earlier workspaces lay in, at the same
    place or beside it, with small tensors written over parts of it in between."""
    import torch

    b, E, I = 64, 256, 1024
    rng, dev, ref, _ = _layer(api, 8700, E, I, b, 0.5)
    held = []
    for n in range(60):
        T = int(rng.integers(1, 9))
        x = synth.gauss_bf16(rng, (T, E), 1.0)
        y = api.sparse_mlp(*dev, to_dev(x))
        torch.cuda.synchronize()
        check_close(y.cpu().numpy().T, orc.mlp(*ref, x), f"call {n} T={T}")
        held = [t for t in held if rng.random() < 0.5]
        held += [torch.randint(0, 1 << 30, (int(rng.integers(1, 2000)),), device="cuda:0") for _ in range(4)]


@pytest.mark.parametrize("b,T", [(64, 1), (64, 4), (64, 16), (128, 2), (128, 16)])
def test_replays_after_the_control_block_was_written_over(api, b, T):
    """Something else is written over the start of the workspace between two replays of a recorded call, so that the
    hand-over state is set up afresh, while the words or slots and H of the replay before stay: no replay takes them."""
    import torch

    E, I = 4 * b, 16 * b
    rng, dev, ref, _ = _layer(api, 8600 + b + T, E, I, b, 0.5)
    ws = torch.randint(0, 256, (api.mlp_workspace_bytes(*dev, T),), dtype=torch.uint8, device="cuda:0")
    xs = to_dev(synth.gauss_bf16(rng, (T, E), 1.0))
    y = torch.empty((T, E), device="cuda:0")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.sparse_mlp(*dev, xs, out=y, ws=ws)
    for rep, written in enumerate((0, 8, 512, 2048, 8448, 0, 8, 8, 4096)):
        ws[:written].random_(0, 256)
        x = synth.gauss_bf16(rng, (T, E), 1.0)
        xs.copy_(to_dev(x))
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        check_close(y.cpu().numpy().T, orc.mlp(*ref, x), f"replay {rep} after {written} bytes, b={b} T={T}")
        assert api.sparse_mlp_status(dev[0], T, ws) == 0


@pytest.mark.parametrize("b,T", [(64, 3), (128, 1), (64, 40), (128, 16), (128, 24)])
def test_a_wait_that_expires_gives_nan_rows_and_a_status(api, b, T):
    """Forced from the host: the producers never publish, the consumers poll 20 times and give up.  Every
    workgroup exits normally; the rows of Y that depended on H are NaN, rows of empty block rows are zeros,
    the status word says 1 and is cleared by reading it; the next ordinary call on the same workspace is right."""
    import torch

    E, I = 4 * b, 6 * b
    rng, dev, ref, masks = _layer(api, 8300 + b, E, I, b, 0.5)
    L = api.lib()
    ws = torch.empty(max(api.mlp_workspace_bytes(*dev, T), 256), dtype=torch.uint8, device="cuda:0")
    x = synth.gauss_bf16(rng, (T, E), 1.0)
    xd = to_dev(x)
    y = torch.full((T, E), 7.0, device="cuda:0")
    vg, vu, vd = (p.view() for p in dev)
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    rc = L.blast_sparse_mlp_handover_test(C.byref(vg), C.byref(vu), C.byref(vd), C.c_void_p(xd.data_ptr()), E,
                                          api.TOKEN_MAJOR, T, api.ACT["silu"], C.c_void_p(y.data_ptr()), E, api.F32,
                                          C.c_void_p(ws.data_ptr()), ws.numel(), stream, 20, 1)
    assert rc == 0
    torch.cuda.synchronize()
    yh = y.cpu().numpy()
    has_blocks = masks[2].sum(axis=1) > 0  # per block row of the down projection
    for br in range(E // b):
        rows = yh[:, br * b:(br + 1) * b]
        if has_blocks[br]:
            assert np.isnan(rows).all(), f"block row {br}: waited-for rows must be NaN"
        else:
            assert not rows.any(), f"block row {br}: nothing to wait for, zeros"
    assert api.sparse_mlp_status(dev[0], T, ws) == 1
    assert api.sparse_mlp_status(dev[0], T, ws) == 0  # cleared by the read
    # argument check of the diagnostic call
    assert L.blast_sparse_mlp_handover_test(C.byref(vg), C.byref(vu), C.byref(vd), C.c_void_p(xd.data_ptr()), E,
                                            api.TOKEN_MAJOR, T, api.ACT["silu"], C.c_void_p(y.data_ptr()), E, api.F32,
                                            C.c_void_p(ws.data_ptr()), ws.numel(), stream, 0, 1) == -1
    # the workspace is fine afterwards
    y2 = api.sparse_mlp(*dev, xd, ws=ws)
    torch.cuda.synchronize()
    check_close(y2.cpu().numpy().T, orc.mlp(*ref, x), "after a timed-out launch")
    assert api.sparse_mlp_status(dev[0], T, ws) == 0
