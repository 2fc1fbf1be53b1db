"""The bf16 table forward at the sizes where its tiling can go wrong, and with
boundaries at the edges of what its table holds, and the full-range kernel
with boundaries that table does not hold, against the oracle: codes bit-exact,
y within one unit in the last place.  Sizes: one
element, both sides of a tile and of a workgroup's 32 tiles (or 8
workgroups' 16), and both sides of the size where the launch shape changes."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2202_00441_amd as P
from parity import OACT, THREADS, check_exact, check_y, download, download_codes, upload

pytestmark = pytest.mark.gpu

WG = 32 * 512
LARGE = 1 << 25
SIZES = [1, 511, 512, 513, WG - 1, WG, WG + 513, 9 * WG + 7,
         LARGE - 1, LARGE, LARGE + 65536 + 1, LARGE + 3 * 512 + 5]


def _check(act, bits, s, v, x_bits, symmetric=False, label=""):
    n = x_bits.size
    flags = P.FLAG_TABLE_FWD | (P.FLAG_SYMMETRIC if symmetric else 0)
    table = P.Table.from_values(P.ACTS[act], bits, s, v, flags=flags)
    print(f"[tab] {act} b{bits} n={n} sym={symmetric} {label}", flush=True)
    guard = 64
    x = upload(x_bits, "bf16")
    y = torch.full((n + guard,), -7.0, dtype=torch.bfloat16, device="cuda")
    words = P.packed_words(n, bits)
    codes = torch.full((words + guard,), -7, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert P.fwd_raw(table, P.BF16, x.data_ptr(), y.data_ptr(), codes.data_ptr(), n, stream) == 0
    torch.cuda.synchronize()
    assert (y[n:] == -7.0).all() and (codes[words:] == -7).all(), "written past the end"
    y_ref, c_ref = O.fwd(OACT[act], O.BF16, bits, np.float32(s), x_bits, symmetric=symmetric, threads=THREADS)
    check_exact(download_codes(codes[:words]), c_ref, f"{label} codes")
    check_y(download(y[:n], "bf16"), y_ref, "bf16", f"{label} y")


def _levels(bits):
    k = 1 << bits
    return [(-2.4 + 4.8 * (m + 1) / k) for m in range(k - 1)], [0.1 * m for m in range(k)]


# the large shape by two activations, the smaller sizes by four
CASES = [(a, b, n) for a, b in (("gelu", 3), ("selu", 2), ("tanh", 4), ("softplus", 1)) for n in SIZES
         if n < LARGE - 1 or a in ("gelu", "selu")]


@pytest.mark.parametrize("act,bits,n", CASES)
def test_sizes(act, bits, n):
    s, v = _levels(bits)
    rng = np.random.default_rng(n % 1000003)
    x = (rng.standard_normal(n, dtype=np.float32) * 3).view(np.uint32)
    bits16 = (x >> 16).astype(np.uint16)
    if n > 600:                                  # NaNs of both signs and infinities, wherever a wave may hold them
        at = rng.integers(0, n, 40)
        bits16[at] = np.resize(np.array([0x7FC1, 0xFFC1, 0x7F80, 0xFF80, 0x7F81, 0x8000], np.uint16), 40)
    _check(act, bits, s, v, bits16, label=f"n={n}")


@pytest.mark.parametrize("act", ["gelu", "silu", "sigmoid", "tanh", "relu", "selu", "softplus"])
@pytest.mark.parametrize("symmetric", [False, True])
def test_boundaries_at_the_edges(act, symmetric):
    # held by the table (0, ordinary sizes) and not held (tiny, huge): either
    # way every pattern's code is the oracle's
    pats = np.random.default_rng(3).permutation(np.arange(1 << 16, dtype=np.uint32).astype(np.uint16))
    tiny, huge = 1e-39, 3e38
    sets = [[0.0], [-0.0], [tiny], [-tiny], [huge], [-huge], [1e-3], [-1e-3], [15.0], [-15.0], [15.9375], [127.5],
            [0.001953125], [-0.001953125]]
    for s in sets:
        _check(act, 1, s, [0.25, 0.75], pats, symmetric, label=f"s={s}")
    _check(act, 2, [-1.5, 0.0, 1.5], [0.0, 0.25, 0.5, 1.0], pats, symmetric, label="around 0")


# the last size: 4096 groups of 4 tiles, two for each of the grid's waves on 256
# compute units, two leftover tiles and a partial one
@pytest.mark.parametrize("n", [1, 511, 513, 2 * 65536 + 77, (1 << 23) + 1234])
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("symmetric", [False, True])
def test_full_range_kernel(bits, symmetric, n):
    s, v = _levels(bits)
    x = np.random.default_rng(n + bits).integers(0, 1 << 16, n).astype(np.uint16)      # every kind of pattern
    act = ("gelu", "softplus", "tanh")[bits - 2]
    if symmetric:
        s = [abs(s[0]) / len(s) * (m + 1) for m in range(len(s))]
    tiny = sorted([1e-39] + [b for b in s if abs(b) > 1e-3])[:len(s)]
    huge = sorted(s[1:] + [3e38])
    for held_out in (tiny, huge):
        held_out = held_out + [4.0 + m for m in range(len(s) - len(held_out))]
        _check(act, bits, held_out, v, x, symmetric, label=f"not held, n={n}")


@pytest.mark.slow
def test_forward_in_parts():
    # past 2^34 elements the per-element forward is launched in parts: bf16,
    # in place (37 GB resident), checked around the seam, at the end and at random
    n = (1 << 34) + 12345
    bits, s = 1, [0.25]
    table = P.Table.from_values(P.ACTS["relu"], bits, s, [0.0, 1.0])
    print(f"[parts] n={n}", flush=True)
    x = torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(3))
    rng = np.random.default_rng(4)
    idx = np.unique(np.concatenate([np.arange((1 << 34) - 2048, (1 << 34) + 2048), np.arange(n - 3000, n),
                                    rng.integers(0, n, 100000)]))
    it = torch.from_numpy(idx).cuda()
    xs = x[it].view(torch.int16).cpu().numpy().view(np.uint16)
    _, codes = P.fwd(table, x, y=x)
    torch.cuda.synchronize()
    ys = x[it].view(torch.int16).cpu().numpy().view(np.uint16)
    y_ref, _, idx_ref = O.fwd(OACT["relu"], O.BF16, bits, np.float32(s), xs, want_idx=True)
    check_y(ys, y_ref, "bf16", "y sampled")
    words = codes[torch.from_numpy(idx // 32).cuda()].cpu().numpy().view(np.uint32)
    got = (words >> (idx % 32).astype(np.uint32)) & 1
    check_exact(got.astype(np.int64), np.asarray(idx_ref).astype(np.int64), "codes sampled")
    del x, codes
    torch.cuda.empty_cache()


@pytest.mark.slow
@pytest.mark.parametrize("dt,bits", [("bf16", 3), ("f32", 1)])
def test_both_directions_in_parts(dt, bits):
    # past 2^35 elements every direction needs several launches (one holds fewer
    # than 2^32 threads, 64 for 512 elements): the forward and then the backward,
    # each in place (up to 142 GB resident), checked around the parts' seams, at
    # the end and at random
    n, part = (1 << 35) + 12345, 1 << 34
    s = [0.25] if bits == 1 else [-1.5, -1.0, -0.5, 0.0, 0.5, 1.0, 1.5]
    v = [0.25 * (m + 1) for m in range(1 << bits)]
    table = P.Table.from_values(P.ACTS["relu"], bits, s, v)
    kind, size = (torch.int32, np.uint32) if dt == "f32" else (torch.int16, np.uint16)
    tdt, odt = (torch.float32, O.F32) if dt == "f32" else (torch.bfloat16, O.BF16)
    print(f"[parts] {dt} n={n} bits={bits}", flush=True)
    x = torch.empty(n, dtype=tdt, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(5)
    for at in range(0, n, 1 << 30):
        x[at:at + (1 << 30)].normal_(generator=gen)
    rng = np.random.default_rng(6)
    idx = np.unique(np.concatenate([np.arange(k * part - 2048, k * part + 2048) for k in (1, 2)] +
                                   [np.arange(n - 3000, n), np.arange(2048), rng.integers(0, n, 100000)]))
    it = torch.from_numpy(idx).cuda()
    sample = lambda: x[it].view(kind).cpu().numpy().view(size)  # noqa: E731
    xs = sample()
    _, codes = P.fwd(table, x, y=x)
    ys = sample()
    y_ref, _, idx_ref = O.fwd(OACT["relu"], odt, bits, np.float32(s), xs, want_idx=True)
    idx_ref = np.asarray(idx_ref).astype(np.int64)
    check_y(ys, y_ref, dt, "y sampled")
    got = np.zeros(idx.size, np.int64)
    for b in range(bits):                       # a code may lie across two words
        at = bits * idx + b
        words = codes[torch.from_numpy(at // 32).cuda()].cpu().numpy().view(np.uint32)
        got |= ((words >> (at % 32).astype(np.uint32)) & 1).astype(np.int64) << b
    check_exact(got, idx_ref, "codes sampled")
    P.bwd(table, x, codes, grad_in=x)
    y32 = ys.view(np.float32) if dt == "f32" else (ys.astype(np.uint32) << 16).view(np.float32)
    want = y32 * np.float32(v)[idx_ref]
    want = want.view(np.uint32) if dt == "f32" else O.round_array(O.BF16, want.astype(np.float64))
    check_exact(sample(), want, "grad_in sampled")
    del x, codes
    torch.cuda.empty_cache()
