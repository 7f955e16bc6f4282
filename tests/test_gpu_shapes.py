"""Stage shapes at the edges of the kernels' tiles and dispatch rules: every
task of a few mini-batches against the oracle's recomputation of it, in both
metrics and at the bounds of the stepwise tests."""
import pytest

import synth
from stepwise import run_stepwise

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _run(kind, dtype, head, batch, layers, dims, lr, k=1, N=3, steps=5):
    spec = synth.StageSpec(kind, dtype, head, k, N, batch, layers, dims, lr, 0.9)
    name = f"{kind}-{dtype}-{head}-b{batch}-l{layers}-{'x'.join(map(str, dims))}"
    print(f"[shapes] {name}", flush=True)
    # forced: float32 masks flip too where a unit lies within a rounding of zero
    worst = run_stepwise(synth.Workload(name, (spec,), steps), steps, torch, forced=True)
    print(f"[shapes] {name}: {worst.report()}", flush=True)


# dims (in, out, hidden). One value in one layer; 32 x 32 tiles with remainders
# and K below one wave's share; the same with leading dimensions and extents
# that no 16-byte load fits; the short kernel's largest K; products past it by
# three (ragged 64 x 64 tiles, element loads), and a weight gradient past the
# short kernel's tile limit with vector loads.
@pytest.mark.parametrize("head,batch,layers,dims", [
    ("none", 1, 1, (1, 1, 1)), ("ce", 31, 2, (64, 10, 36)), ("ce", 33, 2, (131, 7, 65)),
    ("none", 128, 2, (1024, 256, 1024)), ("none", 67, 2, (1027, 259, 514)), ("ce", 130, 2, (516, 1000, 1036)),
])
def test_float32_products(head, batch, layers, dims):
    _run("fc", "fp32", head, batch, layers, dims, 1e-2)


# dims (H, H, T[, vocab]): H no multiple of 32 (short last k fragment) nor of 16
# (short last unit block of the backward); batches past one row block of either
# direction with remainders; ten whole row blocks and one row past them.
@pytest.mark.parametrize("head,batch,dims", [
    ("none", 1, (8, 8, 3, 8)), ("ce", 33, (72, 72, 4, 24)), ("none", 100, (40, 40, 3, 8)), ("none", 65, (1032, 1032, 3, 8)),
    ("none", 320, (512, 512, 3, 8)), ("none", 321, (512, 512, 3, 8)),
])
def test_lstm_steps(head, batch, dims):
    _run("reslstm", "bf16", head, batch, 2, dims, 1e-2)


# bf16 products: one tile and few tiles of ragged M, N and K; K in several slices
# (convolutions); class counts that are no multiple of 8 (element
# stores) and float32 scores of ragged row counts; a convolution grid inside
# the 8-wave range (7/8 of the CUs) with a ragged last row tile.
@pytest.mark.parametrize("kind,head,batch,layers,dims", [
    ("fc", "ce", 50, 2, (1024, 16, 520)), ("fc", "none", 129, 2, (136, 264, 1160)),
    ("conv3x3", "ce", 10, 1, (160, 168, 10, 10, 10)), ("conv3x3", "none", 33, 2, (40, 72, 7, 9)),
    ("conv3x3", "none", 113, 1, (64, 512, 8, 8)), ("bottleneck", "ce", 10, 1, (264, 72, 7, 7, 6)),
    ("transformer", "ce", 3, 1, (64, 1, 72, 40, 1000)),
])
def test_bf16_products(kind, head, batch, layers, dims):
    _run(kind, "bf16", head, batch, layers, dims, 1e-4)


# dims (d, heads, ffn, S[, vocab]): one short score tile, one whole tile at head
# dimension 32, one row past a tile, whole tiles, and a head dimension that
# keeps the batched-GEMM form.
@pytest.mark.parametrize("batch,dims", [
    (2, (64, 1, 72, 8, 8)), (2, (64, 2, 72, 128, 8)), (3, (128, 2, 136, 136, 8)), (1, (128, 4, 136, 256, 8)),
    (2, (128, 2, 136, 328, 8)), (2, (64, 4, 72, 48, 8)),
])
def test_attention_lengths(batch, dims):
    _run("transformer", "bf16", "none", batch, 1, dims, 1e-3)


@pytest.mark.parametrize("dims", [(64, 2, 72, 136), (128, 2, 136, 40)])
def test_stash_probabilities(dims):
    """read_stash ids 1 and 2 hold the softmax probabilities of the stashed
    qkv. Bounds: float32 scores of up to 64 products and the exponential's own
    error, 2e-5 of the largest probability; bf16 rounding, 2^-8 of each."""
    import numpy as np

    from paper_1809_02839_amd import native
    d, heads, _, S = dims
    B, dh = 2, d // heads
    spec = synth.StageSpec("transformer", "bf16", "none", 0, 1, B, 1, dims, 1e-3, 0.9)
    st = native.Stage(native.desc_from_spec(spec), synth.initial_params(spec), torch.cuda.current_stream())
    x = torch.from_numpy(synth.stage_input(spec, 0) * 50).cuda().bfloat16()
    y = torch.empty_like(x)
    st.forward(0, x, y)
    raw = {i: st.read_stash(0, i) for i in (0, 1, 2)}
    bf = lambda a: (a.view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)  # noqa: E731
    q, k, _ = bf(raw[0]).reshape(B, S, 3, heads, dh).transpose(2, 0, 3, 1, 4)
    z = q @ k.transpose(0, 1, 3, 2) / np.sqrt(dh)
    p = np.exp(z - z.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    got = raw[1].view(np.float32).reshape(p.shape)
    assert np.max(np.abs(got - p)) <= 2e-5 * p.max()
    assert np.max(np.abs(bf(raw[2]).reshape(p.shape) - got) / got) <= 2.0 ** -8
    st.destroy()


@pytest.mark.parametrize("S,hidden", [(40, 32), (136, 32), (136, 131)])
def test_scores_of_minus_infinity(S, hidden):
    """Scores that overflow to -infinity over the first `hidden` keys (whole
    column groups, a whole tile) weigh nothing: the context is the mean of the
    other keys' values. bf16 rounding of P, of v and of the result: 3 x 2^-8
    of the values' mean magnitude."""
    import numpy as np

    from paper_1809_02839_amd import native
    d, B = 64, 1
    spec = synth.StageSpec("transformer", "bf16", "none", 0, 1, B, 1, (d, 1, 72, S), 1e-3, 0.9)
    W = synth.initial_params(spec)
    w, b = np.zeros((3 * d, d), np.float32), np.zeros(3 * d, np.float32)
    b[0] = 1e20                  # q = (1e20, 0, ...)
    w[d, 0] = -3e20              # k = (-3e20 x0, 0, ...)
    w[2 * d + 1, 1] = 1.0        # v = (0, x1, 0, ...)
    W[:w.size], W[w.size:w.size + b.size] = w.ravel(), b
    x = torch.zeros(B, S, d)
    x[:, :hidden, 0] = 1.0
    x[:, :, 1] = 1.0 + torch.arange(S) % 7
    st = native.Stage(native.desc_from_spec(spec), W, torch.cuda.current_stream())
    xg = x.cuda().bfloat16()
    st.forward(0, xg, torch.empty_like(xg))
    ctx = (st.read_stash(0, 3).view(np.uint16).astype(np.uint32) << 16).view(np.float32).reshape(B, S, d)
    st.destroy()
    mean = float(x[0, hidden:, 1].mean())
    assert np.max(np.abs(ctx[..., 1] - mean)) <= 3 * 2.0 ** -8 * mean


# Filter gradients left in K-slice planes for the update: 11 and 3 slices by
# the rule at these pixel counts. The planes lie in memory that held NaN before,
# so one that the launch did not write shows.
@pytest.mark.parametrize("batch,dims", [(32, (128, 128, 14, 14)), (11, (104, 328, 12, 7))])
def test_filter_gradient_planes(batch, dims):
    torch.cuda.empty_cache()
    dirty = torch.full((1 << 28,), float("nan"), device="cuda")
    torch.cuda.synchronize()
    del dirty
    torch.cuda.empty_cache()
    _run("conv3x3", "bf16", "none", batch, 1, dims, 1e-4)


# A bottleneck's forward: 2 slices (1 x 1, K = 1920) and 5 (3 x 3, K = 4320), not
# the 3 of the time model for the first; a fully connected layer: 5 (K = 4104),
# not 13. Another order moves v by more than two versions may differ.
@pytest.mark.parametrize("kind,batch,dims,floats", [
    ("bottleneck", 15, (1920, 480, 8, 8), 960 * 480 * (2 + 5)), ("fc", 50, (4104, 264, 264), 50 * 264 * 5),
])
def test_products_keep_their_slices(kind, batch, dims, floats):
    from paper_1809_02839_amd import native
    spec = synth.StageSpec(kind, "bf16", "none", 0, 1, batch, 1, dims, 1e-6, 0.9)
    st = native.Stage(native.desc_from_spec(spec), synth.initial_params(spec), torch.cuda.current_stream())
    x = torch.from_numpy(synth.stage_input(spec, 0)).cuda().bfloat16()
    y = torch.empty(spec.output_shape(), dtype=torch.bfloat16, device="cuda")
    st.profile(True)
    st.forward(0, x, y)
    torch.cuda.synchronize()
    planes = sum(s["extra_bytes_total"] for n, s in st.profile_read().items() if n.startswith("gemm_bf16"))
    st.destroy()
    assert planes == 4 * floats


# Either side of the rule's lines: the largest batch of the fused steps and the
# first of a GEMM and a cell launch per step, by rows H^2 and by B H.
@pytest.mark.parametrize("batch,H,fused", [
    (512, 512, True), (513, 512, False), (128, 1024, True), (129, 1024, False), (8, 2560, True), (17, 2560, False),
    (1024, 256, True), (1025, 256, False),
])
def test_lstm_rule(batch, H, fused):
    from paper_1809_02839_amd import native
    spec = synth.StageSpec("reslstm", "bf16", "none", 0, 1, batch, 1, (H, H, 2, 8), 1e-2, 0.9)
    st = native.Stage(native.desc_from_spec(spec), synth.initial_params(spec), torch.cuda.current_stream())
    x = torch.from_numpy(synth.stage_input(spec, 0)).cuda().bfloat16()
    y, dx = torch.empty_like(x), torch.empty_like(x)
    st.profile(True)
    st.forward(0, x, y)
    st.backward(0, torch.ones_like(x) / x.numel(), dx)
    torch.cuda.synchronize()
    names = set(st.profile_read())
    st.destroy()
    assert {"lstm_step", "lstm_step_bwd"} <= names if fused else {"lstm_cell", "lstm_cell_bwd"} <= names
    if H == 512:
        _run("reslstm", "bf16", "none", batch, 1, (H, H, 2, 8), 1e-2, steps=3)


# Products on the 64 x 64 tiles in every operand mode: whole tiles with 16-byte
# loads, K in 5 to 16 slices; and sizes that no tile, K step or 16-byte load
# fits, K in 3 to 13 slices of which the last is short (element loads).
@pytest.mark.parametrize("head,batch,dims,vec", [
    ("ce", 128, (3072, 10, 2048), "true"), ("none", 131, (3075, 259, 2051), "false"),
])
def test_float32_tiles(head, batch, dims, vec):
    from paper_1809_02839_amd import native
    spec = synth.StageSpec("fc", "fp32", head, 0, 1, batch, 3, dims, 1e-2, 0.9)
    st = native.Stage(native.desc_from_spec(spec), synth.initial_params(spec), torch.cuda.current_stream())
    x = torch.from_numpy(synth.stage_input(spec, 0)).cuda().float()
    y = torch.empty(batch, dims[1], device="cuda") if head == "none" else None
    lab = torch.zeros(batch, dtype=torch.int32, device="cuda") if head == "ce" else None
    st.profile(True)
    st.forward(0, x, y, lab, torch.zeros(1, device="cuda") if head == "ce" else None)
    st.backward(0, y, torch.empty_like(x))
    torch.cuda.synchronize()
    names = set(st.profile_read())
    st.destroy()
    assert {f"gemm_f32_kernel<{m}, {vec}>" for m in ("0, 0", "0, 3", "3, 3")} <= names, names
    _run("fc", "fp32", head, batch, 3, dims, 1e-2, steps=3)


def _bf(a):
    import numpy as np
    return (a.view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("dims", [(64, 2, 72, 136), (128, 2, 136, 40)])
def test_stash_probabilities_are_the_passes_own(dims):
    """The context is bf16(P) V of the probabilities that read_stash returns
    (bounds: bf16 rounding of each entry and a float32 sum of S terms), and
    reading them launches nothing that the stage's profile counts."""
    import numpy as np

    from paper_1809_02839_amd import native
    d, heads, _, S = dims
    B, dh = 3, d // heads
    spec = synth.StageSpec("transformer", "bf16", "none", 0, 1, B, 1, dims, 1e-3, 0.9)
    st = native.Stage(native.desc_from_spec(spec), synth.initial_params(spec), torch.cuda.current_stream())
    x = torch.from_numpy(synth.stage_input(spec, 0) * 50).cuda().bfloat16()
    st.profile(True)
    st.forward(0, x, torch.empty_like(x))
    before = {k: v["launches"] for k, v in st.profile_read().items()}
    raw = {i: st.read_stash(0, i) for i in (0, 1, 2, 3)}
    assert {k: v["launches"] for k, v in st.profile_read().items()} == before
    st.destroy()
    p = _bf(raw[2]).reshape(B, heads, S, S)
    v = _bf(raw[0]).reshape(B, S, 3, heads, dh)[:, :, 2].transpose(0, 2, 1, 3)
    ctx = _bf(raw[3]).reshape(B, S, heads, dh).transpose(0, 2, 1, 3)
    want, size = p @ v, p @ np.abs(v)
    assert np.all(np.abs(ctx - want) <= 2.0 ** -8 * np.abs(want) + S * 2.0 ** -24 * size)
    f32 = raw[1].view(np.float32).reshape(p.shape)
    assert np.array_equal(_bf(torch.from_numpy(f32).bfloat16().view(torch.int16).numpy()), p)


@pytest.mark.parametrize("S", [56, 264])
def test_exponential_over_its_range(S):
    """Scores from 0 down past the exponential's underflow against float64's
    probabilities. Bounds: two units of 2^-23 for the exponential, one for the
    division and its product, 2^-24 for each of a lane's S / 2 terms of the sum,
    and 2^-126 where float32 has no normal numbers."""
    import numpy as np

    from paper_1809_02839_amd import native
    d, B = 64, 1
    spec = synth.StageSpec("transformer", "bf16", "none", 0, 1, B, 1, (d, 1, 72, S), 1e-3, 0.9)
    W = synth.initial_params(spec)
    w, b = np.zeros((3 * d, d), np.float32), np.zeros(3 * d, np.float32)
    b[0] = 8.0                   # q = (8, 0, ...): score = k0 at scale 1 / 8
    w[d, 0] = 1.0                # k = (x0, 0, ...)
    W[:w.size], W[w.size:w.size + b.size] = w.ravel(), b
    x = torch.zeros(B, S, d)
    x[0, :, 0] = torch.linspace(0.0, -1.0, S) ** 3 * 120.0
    x = x.bfloat16()
    st = native.Stage(native.desc_from_spec(spec), W, torch.cuda.current_stream())
    xg = x.cuda()
    st.forward(0, xg, torch.empty_like(xg))
    p = st.read_stash(0, 1).view(np.float32).reshape(S, S).astype(np.float64)
    st.destroy()
    e = np.exp(x[0, :, 0].double().numpy())
    want = e / e.sum()
    assert np.count_nonzero(want < 2.0 ** -126) >= S // 16 and want.max() > 0.01
    assert np.all(np.abs(p - want) <= (3 + S / 4) * 2.0 ** -23 * want + 2.0 ** -126)


# Either side of the line between the score tiles and the batched GEMMs: past
# 768 positions 88 blocks of 128 rows.
@pytest.mark.parametrize("batch,S,tiles", [(1, 768, True), (1, 776, False), (13, 776, True), (12, 776, False)])
def test_attention_rule(batch, S, tiles):
    from paper_1809_02839_amd import native
    spec = synth.StageSpec("transformer", "bf16", "none", 0, 1, batch, 1, (64, 1, 72, S, 8), 1e-3, 0.9)
    st = native.Stage(native.desc_from_spec(spec), synth.initial_params(spec), torch.cuda.current_stream())
    x = torch.from_numpy(synth.stage_input(spec, 0)).cuda().bfloat16()
    st.profile(True)
    st.forward(0, x, torch.empty_like(x))
    torch.cuda.synchronize()
    names = set(st.profile_read())
    st.destroy()
    assert ("attention_long" in names) == tiles and ("softmax" in names) != tiles, names
    if batch == 1:
        _run("transformer", "bf16", "none", 1, 1, (64, 1, 72, S, 8), 1e-3, steps=3)
