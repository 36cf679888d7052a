"""The kernels for long token loops (128 x 256 tiles; 256 x 128 for int8 column blocks) against
the 128 x 128 kernel, bit for bit.

Steps are tile-local and every kernel sums a tile's products in the same order, so a matrix
large enough for the long-loop kernel must end with the same bits as its row slices stepped one
by one, which are too small for it; the kernel that steps the slices is checked against the
oracle elsewhere.  (bf16 at T = 1025 and fp32 at 1056 are below the rule: the other kernel's.)  Sizes leave remainders on every axis, more tiles than resident workgroups
(a workgroup walks several tiles), and a last chunk of one token.
"""
import pytest
import torch

from gpu_util import HP
from paper_2606_22932_amd import forge

pytestmark = pytest.mark.gpu

D_IN, D_OUT, SLICE = 4104, 8264, 1024      # 17 x 65 tiles of 256 columns x 128 rows; 33 x 33 of 128 x 256


def _gauss(shape, std, gen, dtype=torch.bfloat16):
    return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(dtype)


def _state(kind, rows, gen, d_in=D_IN):
    """State tensors of [rows, d_in] by argument name."""
    shape = (rows, d_in)
    codes = lambda lo, hi: torch.randint(lo, hi, shape, generator=gen, device="cuda", dtype=torch.int8)
    def fp8(signed):         # every finite code, of either sign or none
        c = torch.randint(0, 0x7F, shape, generator=gen, device="cuda", dtype=torch.uint8)
        if signed:
            c |= torch.randint(0, 2, shape, generator=gen, device="cuda", dtype=torch.uint8) << 7
        return c.view(torch.float8_e4m3fn)
    ring = lambda a: torch.tensor([0.0, 0.0, a, a], device="cuda")
    s = {"W": _gauss(shape, 0.02, gen)}
    if kind in ("bf16", "f32", "wfp8_bf16"):
        dt = torch.float32 if kind == "f32" else torch.bfloat16
        s["m"], s["v"] = _gauss(shape, 1e-4, gen, dt), _gauss(shape, 1e-6, gen, torch.float32).abs_().to(dt)
    elif kind in ("i8", "i8r64"):
        sshape = ((rows + 255) // 256, d_in) if kind == "i8" else (rows, (d_in + 63) // 64)
        s["m"], s["v"] = codes(-127, 128), codes(1, 128)
        u = lambda x: torch.rand(sshape, generator=gen, device="cuda").add_(0.5).mul_(x / 127)
        s["ms"], s["vs"] = u(3e-4), u(3e-3 if kind == "i8" else 3e-6)
    else:
        s["m"], s["v"] = fp8(True), fp8(False)
        s["ms"], s["vs"] = ring(3e-4), ring(3e-3)
    if kind.startswith("wfp8"):
        s["W"], s["wr"] = fp8(True), ring(0.06)
    return s


def _step(kind, X, dY, s):
    if kind.startswith("wfp8"):
        forge.forge_linear_step_wfp8(X, dY, s["W"], s["wr"], s["m"], s["v"], s.get("ms"), s.get("vs"), step=100, **HP)
    else:
        forge.forge_linear_step(X, dY, s["W"], s["m"], s["v"], s.get("ms"), s.get("vs"), step=100, **HP)


def _rows(kind, name, t, r0, r1):
    """The part of state tensor `name` that belongs to rows r0..r1 (a ring: all of it)."""
    if t.shape == (4,):
        return t
    if kind == "i8" and name in ("ms", "vs"):
        return t[r0 // 256:(r1 + 255) // 256]
    return t[r0:r1]


def _raw(t):
    """t as integers of its size, which compare NaNs too."""
    return t.view({1: torch.uint8, 2: torch.int16, 4: torch.int32}[t.element_size()])


@pytest.mark.parametrize("kind,T", [("bf16", 1537), ("f32", 1568), ("bf16", 1025), ("f32", 1056), ("i8r64", 513),
                                    ("fp8", 544), ("wfp8_bf16", 545), ("wfp8_fp8", 257), ("i8", 0), ("i8", 1),
                                    ("i8", 70), ("i8", 513)])
def test_long_loop_kernel_equals_row_slices_bitwise(kind, T):
    print("case", kind, T, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    X, dY = _gauss((T, D_IN), 1.0, gen), _gauss((T, D_OUT), 1e-3, gen)
    _whole_equals_slices(kind, X, dY, _state(kind, D_OUT, gen))


@pytest.mark.parametrize("bad", [float("nan"), float("inf")], ids=str)
@pytest.mark.parametrize("kind,T", [("fp8", 544), ("wfp8_fp8", 257), ("i8", 70), ("i8r64", 513)])
def test_long_loop_kernel_passes_nan_and_inf_like_row_slices(kind, T, bad):
    """A NaN or Inf token makes a column of G NaN or infinite, and what a tile holds outside the
    matrix NaN (zero times Inf): maxima pass NaNs by, and take no part of what is outside."""
    print("case", kind, T, bad, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(16)
    X, dY = _gauss((T, D_IN), 1.0, gen), _gauss((T, D_OUT), 1e-3, gen)
    X[T - 1, 17] = X[3, D_IN - 1] = bad
    dY[5, D_OUT - 9] = float("nan")
    whole = _state(kind, D_OUT, gen)
    _whole_equals_slices(kind, X, dY, whole)
    if "fp8" in kind:
        assert bool(torch.isfinite(whole["ms"][0])) == (bad != bad) and float(whole["vs"][0]) > 0


def _whole_equals_slices(kind, X, dY, whole):
    parts = []
    for r0 in range(0, D_OUT, SLICE):
        r1 = min(r0 + SLICE, D_OUT)
        parts.append((r0, r1, {k: _rows(kind, k, t, r0, r1).clone() for k, t in whole.items()}))
    _step(kind, X, dY, whole)
    for r0, r1, s in parts:
        _step(kind, X, dY[:, r0:r1].contiguous(), s)
    torch.cuda.synchronize()
    for k, t in whole.items():
        if t.shape == (4,):        # amax ring: this step's slot is the largest of the slices'
            want = torch.stack([s[k] for _, _, s in parts]).amax(0)
            assert torch.equal(t, want), k
            continue
        for r0, r1, s in parts:
            assert torch.equal(_raw(_rows(kind, k, t, r0, r1)), _raw(s[k])), (k, r0)


@pytest.mark.parametrize("rule,dtype", [("sgd_momentum", torch.float32), ("nadam", torch.bfloat16),
                                        ("muon_accumulate", torch.bfloat16), ("sgd", torch.bfloat16),
                                        ("adagrad", torch.float32), ("rmsprop", torch.bfloat16),
                                        ("lion", torch.bfloat16), ("radam", torch.float32),
                                        ("adamax", torch.bfloat16)])
def test_long_loop_rules_equal_row_slices_bitwise(rule, dtype):
    print("case", rule, dtype, flush=True)
    T = 1543
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    X, dY = _gauss((T, D_IN), 1.0, gen), _gauss((T, D_OUT), 1e-3, gen)
    W = None if rule == "muon_accumulate" else _gauss((D_OUT, D_IN), 0.02, gen)
    ns = forge.OPTIMIZER_STATES[rule]
    st = [_gauss((D_OUT, D_IN), 1e-3, gen, torch.float32).abs_().to(dtype) for _ in range(ns)]
    hp = dict(lr=1e-3, beta1=0.9, beta2=0.99, weight_decay=0.1, step=7)

    def run(dY, W, st):
        forge.forge_linear_step_opt(X, dY, W, *st, optimizer=rule, **hp)

    ranges = [(r, min(r + SLICE, D_OUT)) for r in range(0, D_OUT, SLICE)]
    parts = [(W if W is None else W[a:b].clone(), [t[a:b].clone() for t in st]) for a, b in ranges]
    run(dY, W, st)
    for (a, b), (w, ss) in zip(ranges, parts):
        run(dY[:, a:b].contiguous(), w, ss)
    torch.cuda.synchronize()
    for (a, b), (w, ss) in zip(ranges, parts):
        assert W is None or torch.equal(W[a:b], w), a
        for t, u in zip(st, ss):
            assert torch.equal(t[a:b], u), a


@pytest.mark.parametrize("kind,T", [("bf16", 1552), ("i8", 70), ("i8r64", 520), ("fp8", 520)])
def test_long_loop_group_equals_single_steps_bitwise(kind, T):
    """A group that only together is large enough for the long-loop kernel (int8 columns: with a
    matrix that alone is not); a workgroup goes from one matrix to the next, with its own scales
    and amax ring."""
    print("case", kind, T, flush=True)
    d_in, d_outs = 2056, (7184, 264, 8200)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(13)
    X = _gauss((T, d_in), 1.0, gen)
    mats = [(_gauss((T, d), 1e-3, gen), _state(kind, d, gen, d_in)) for d in d_outs]
    alone = [(dY, {k: t.clone() for k, t in s.items()}) for dY, s in mats]
    forge.forge_linear_step_grouped([(X, dY, s["W"], s["m"], s["v"], s.get("ms"), s.get("vs")) for dY, s in mats],
                                    step=100, **HP)
    for dY, s in alone:
        _step(kind, X, dY, s)
    torch.cuda.synchronize()
    for (_, x), (_, y) in zip(mats, alone):
        for k in x:
            assert torch.equal(_raw(x[k]), _raw(y[k])), k


@pytest.mark.parametrize("T", [33, 97, 192, 224, 2049])
def test_token_loop_forms_are_bitwise_neutral(T):
    """The 128 x 128 kernel's token loop has two forms: with tests in every chunk (less than six
    chunks; T <= 224 or >= 1536 on more than 256 tiles, as the whole here) and without (the slices of
    at most 8 x 33 tiles, 200 at T = 192 and 2049).  Fewer chunks than the ring has stages, one
    more, a ring that goes around, and one form against the other."""
    print("case", T, flush=True)
    d_in, d_out = (3208, 2168) if T in (192, 2049) else (D_IN, D_OUT)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(14)
    X, dY = _gauss((T, d_in), 1.0, gen), _gauss((T, d_out), 1e-3, gen)
    whole = {"W": _gauss((d_out, d_in), 0.02, gen), "m": _gauss((d_out, d_in), 1e-4, gen),
             "v": _gauss((d_out, d_in), 1e-6, gen).abs_()}
    parts = {r0: {k: t[r0:r0 + SLICE].clone() for k, t in whole.items()} for r0 in range(0, d_out, SLICE)}
    _step("bf16", X, dY, whole)
    for r0, s in parts.items():
        _step("bf16", X, dY[:, r0:r0 + SLICE].contiguous(), s)
    torch.cuda.synchronize()
    for r0, s in parts.items():
        for k, t in s.items():
            assert torch.equal(whole[k][r0:r0 + SLICE], t), (k, r0)


@pytest.mark.parametrize("d_in,d_out", [(2056, 4424), (4096, 3272), (4096, 6152), (4104, 1544)], ids=str)
def test_fp32_rasters_are_bitwise_neutral(d_in, d_out):
    """fp32 state with short loops walks its tiles in groups of 4 tile rows (here 35, a remainder of
    3), in one group (26 rows of a 4096 wide matrix), and by the shape rule (49 and 13 rows): every
    tile once, whatever the order."""
    print("case", d_in, d_out, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(15)
    X, dY = _gauss((33, d_in), 1.0, gen), _gauss((33, d_out), 1e-3, gen)
    whole = {"W": _gauss((d_out, d_in), 0.02, gen), "m": _gauss((d_out, d_in), 1e-4, gen, torch.float32),
             "v": _gauss((d_out, d_in), 1e-6, gen, torch.float32).abs_()}
    parts = {r0: {k: t[r0:r0 + 896].clone() for k, t in whole.items()} for r0 in range(0, d_out, 896)}
    _step("f32", X, dY, whole)
    for r0, s in parts.items():
        _step("f32", X, dY[:, r0:r0 + 896].contiguous(), s)
    torch.cuda.synchronize()
    for r0, s in parts.items():
        for k, t in s.items():
            assert torch.equal(whole[k][r0:r0 + 896], t), (k, r0)
