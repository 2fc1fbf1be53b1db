"""Short launches: the partial tile at the end of a tensor at every kind of
remainder, against the oracle, and its cost in a replayed stack of layers."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2202_00441_amd as P
from parity import (ODT, OACT, THREADS, check_exact, check_y, download, download_codes, golden_table, torch_dtype,
                    upload)

pytestmark = pytest.mark.gpu

GUARD = 64


def _bits(dt, n, seed):
    x = np.random.default_rng(seed).standard_normal(n, dtype=np.float32) * 3
    if dt == "f32":
        return x.view(np.uint32)
    return x.astype(np.float16).view(np.uint16) if dt == "f16" else (x.view(np.uint32) >> 16).astype(np.uint16)


def check_guarded(key, dt, n, flags=0):
    """fwd and bwd into buffers with guard elements behind them."""
    spec, table = golden_table(key)
    table = table.with_flags(flags)
    bits = spec["bits"]
    print(f"[small] {key} {dt} n={n} flags={flags}", flush=True)
    xb, gb = _bits(dt, n, n), _bits(dt, n, n + 1)
    x, g = upload(xb, dt), upload(gb, dt)
    y, gin = (torch.full((n + GUARD,), -7.0, dtype=torch_dtype(dt), device="cuda") for _ in range(2))
    words = P.packed_words(n, bits)
    codes = torch.full((words + GUARD,), -7, dtype=torch.int32, device="cuda")
    P.fwd(table, x, y[:n], codes)
    P.bwd(table, g, codes, gin[:n])
    torch.cuda.synchronize()
    assert (y[n:] == -7.0).all() and (gin[n:] == -7.0).all() and (codes[words:] == -7).all(), "past the end"
    s = np.float32([float.fromhex(h) for h in spec["s"]])
    v = np.float32([float.fromhex(h) for h in spec["v"]])
    y_ref, c_ref = O.fwd(OACT[spec["act"]], ODT[dt], bits, s, xb, symmetric=bool(spec.get("symmetric")),
                         threads=THREADS)
    check_exact(download_codes(codes[:words]), c_ref, "codes")
    check_y(download(y[:n], dt), y_ref, dt)
    check_exact(download(gin[:n], dt), O.bwd(ODT[dt], bits, v, gb, c_ref, threads=THREADS), "grad_in")


@pytest.mark.parametrize("rest", [1, 2, 7, 8, 9, 255, 256, 257, 263, 504, 511])
@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_partial_tile(bits, dt, rest):
    for n in (rest, 5 * 512 + rest):
        check_guarded(f"gelu_bf16_lm_ffn_16x2048x8192/b{bits}", dt, n)
        if dt != "f32":
            check_guarded(f"gelu_bf16_lm_ffn_16x2048x8192/b{bits}", dt, n, P.FLAG_TABLE_FWD)


# both sides of the fp32 small kernels' limit (12 tiles)
@pytest.mark.parametrize("key", ["gelu3_f32_1m/b3", "sigmoid4_f32_odd_67108863/b4", "sigmoid4_f32_odd_67108863/b4/sym",
                                 "gelu_bf16_lm_ffn_16x2048x8192/b1", "silu2_f16_resnet_64x256x56x56/b2"])
def test_short_fp32_launches(key):
    for n in (1, 511, 512, 2048, 2049, 6143, 6144, 6145):
        check_guarded(key, "f32", n)


def _stack(table, n, dt, layers):
    """A graph of the forwards and then the backwards of `layers` layers."""
    sets = []
    for _ in range(layers):
        x = torch.randn(n, device="cuda").to(torch_dtype(dt))
        sets.append((x, torch.empty_like(x), torch.empty_like(x),
                     torch.empty(P.packed_words(n, table.bits), dtype=torch.int32, device="cuda")))

    def run():
        for x, y, _, codes in sets:
            P.fwd(table, x, y, codes)
        for x, _, gin, codes in reversed(sets):
            P.bwd(table, x, codes, gin)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    return graph, sets


def _us(graph, replays=100):
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record()
    for _ in range(replays):
        graph.replay()
    end.record()
    end.synchronize()
    return start.elapsed_time(end) * 1e3 / replays


@pytest.mark.parametrize("act,bits,dt", [("sigmoid", 4, "f32"), ("gelu", 3, "bf16"), ("silu", 2, "f16")])
def test_a_ragged_stack_takes_no_longer_than_a_whole_one(act, bits, dt):
    # 12 elements short of a whole tile.  Handled element after element that
    # tile made the stack 1.4 to 1.5 times as long; with its loads in
    # flight together it is within 1.1.
    table = P.fit_table(act, bits, P.Weight(P.W_NORMAL, -10.0, 10.0), 1000)
    whole, ragged = _stack(table, 66 * 512, dt, 12), _stack(table, 66 * 512 - 12, dt, 12)
    times = [(_us(whole[0]), _us(ragged[0])) for _ in range(7)][1:]
    a, b = min(t[0] for t in times), min(t[1] for t in times)
    print(f"[small] {act} {dt} whole {a:.1f} us, ragged {b:.1f} us", flush=True)
    assert b < 1.25 * a


def test_sizes_no_memory_holds_are_refused():
    # nothing is launched: the size is refused on the host
    table = P.fit_table("gelu", 3, P.Weight(P.W_NORMAL, -10.0, 10.0), 1000).with_flags(P.FLAG_ELEMENT_FWD)
    b = torch.zeros(4096, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for n in (1 << 38, 1 << 62):
        for dt in (P.F32, P.F16, P.BF16):
            for f in (P.fwd_raw, P.bwd_raw):
                assert f(table, dt, b.data_ptr(), b.data_ptr(), b.data_ptr(), n, stream) == -8
    torch.cuda.synchronize()
