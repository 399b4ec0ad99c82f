"""Windowed layers (only the last W tokens of each request move) through the
C ABI vs the CPU oracle, bit for bit: reduced workloads element-wise, and the
mixed-kind gpt-oss-120b shape at full size in the benchmark's launch
configuration (sampled layers vs the oracle, every layer by round trip)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, to_dev, to_host
from paper_2607_28633_amd.workloads import (device_dst_prefill, device_src_pool, host_dst_prefill,
                                            host_src_pool, make_workload)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tk():
    from paper_2607_28633_amd import topkv
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return topkv


def _scaled(name, div, **kw):
    base = make_workload(name)
    return make_workload(name, seq_lens=np.maximum(base.seq_lens // div, 1), **kw)


CASES = {
    "tiny-w1": (lambda: make_workload("tiny", seq_lens=[64, 48, 33, 17, 0, 1]), 1),
    "tiny-w17-p48": (lambda: make_workload("tiny", seq_lens=[64, 48, 33, 17, 0, 1], dst_page_size=48), 17),
    "tiny-w40-p5": (lambda: make_workload("tiny", dst_page_size=5), 40),
    "mla-div16-w128": (lambda: _scaled("deepseek-v3-mla", 16, num_layers=2), 128),
    "reblock-div32-w1000": (lambda: _scaled("reblock-70b", 32, num_layers=2, phys_layers=2), 1000),
    "gpt-oss-div8-w128": (lambda: _scaled("gpt-oss-120b", 8, num_layers=2), 128),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_window_parity(tk, case):
    make, W = CASES[case]
    wl = make()
    say(f"[window] {case}: W={W} {wl.describe()}")
    src_h, dst_h = host_src_pool(wl), host_dst_prefill(wl)
    src, dst = to_dev(src_h), to_dev(dst_h)
    bt, bt2, lens = to_dev(wl.block_tables), to_dev(wl.dst_block_tables), to_dev(wl.seq_lens)
    nbytes = tk.topkv_packed_window_bytes(src, wl.seq_lens, W)
    assert nbytes == oracle.packed_layer_elems(wl.planes, wl.num_heads, wl.head_dim, wl.seq_lens, W) * wl.elem_bytes
    want_dst = dst_h.copy()
    for layer in range(wl.num_layers):
        slab = layer % wl.phys_layers
        packed = torch.full((nbytes // wl.elem_bytes + 32,), -9, dtype=src.dtype, device="cuda")
        tk.topkv_pack_layer_window(src, slab, wl.num_reqs, bt, bt.shape[1], lens, W, packed, dst_bytes=nbytes)
        tk.topkv_unpack_layer_window(packed, dst, slab, wl.num_reqs, bt2, bt2.shape[1], lens, W, src_bytes=nbytes)
        torch.cuda.synchronize()
        got = to_host(packed)
        want = oracle.pack_layer(src_h, slab, wl.block_tables, wl.seq_lens, window=W)
        assert np.array_equal(got[:want.size], want), f"{case} layer {layer}: windowed pack differs"
        assert (got[want.size:].view(np.int16) == -9).all(), f"{case}: write past the batch"
        oracle.unpack_layer(want, want_dst, slab, wl.dst_block_tables, wl.seq_lens, window=W)
        assert np.array_equal(to_host(dst)[slab], want_dst[slab]), f"{case} layer {layer}: windowed unpack differs"


def test_window_zero_is_the_batched_call(tk):
    wl = make_workload("tiny")
    src = to_dev(host_src_pool(wl))
    bt, lens = to_dev(wl.block_tables), to_dev(wl.seq_lens)
    nbytes = tk.topkv_packed_layer_bytes(src, wl.seq_lens)
    assert tk.topkv_packed_window_bytes(src, wl.seq_lens, 0) == nbytes
    a = torch.zeros(nbytes // 2, dtype=torch.int16, device="cuda")
    b = torch.ones_like(a)
    tk.topkv_pack_layer_window(src, 1, wl.num_reqs, bt, bt.shape[1], lens, 0, a)
    tk.topkv_pack_layer_batched(src, 1, wl.num_reqs, bt, bt.shape[1], lens, b)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_gpt_oss_fullsize(tk):
    """36 layers alternating 128-token windows and full attention, 32 requests."""
    wl = make_workload("gpt-oss-120b")
    say(f"[window] gpt-oss-120b full size: {wl.describe()}")
    src, dst = device_src_pool(wl), device_dst_prefill(wl)
    bt, bt2, lens = to_dev(wl.block_tables), to_dev(wl.dst_block_tables), to_dev(wl.seq_lens)
    full = tk.topkv_packed_layer_bytes(src, wl.seq_lens)
    packed = torch.empty(full // 2, dtype=torch.int16, device="cuda")
    again = torch.empty_like(packed)
    for layer in range(wl.num_layers):
        W = wl.window(layer)
        nb = tk.topkv_packed_window_bytes(src, wl.seq_lens, W)
        if layer in (0, 1, wl.num_layers - 1):
            torch.cuda.synchronize()
            src_h, dst_before = to_host(src[layer])[None], to_host(dst[layer])[None]
        tk.topkv_pack_layer_window(src, layer, wl.num_reqs, bt, bt.shape[1], lens, W, packed, dst_bytes=nb)
        tk.topkv_unpack_layer_window(packed, dst, layer, wl.num_reqs, bt2, bt2.shape[1], lens, W, src_bytes=nb)
        tk.topkv_pack_layer_window(dst, layer, wl.num_reqs, bt2, bt2.shape[1], lens, W, again, dst_bytes=nb)
        assert torch.equal(packed[:nb // 2], again[:nb // 2]), f"layer {layer}: round trip differs"
        if layer in (0, 1, wl.num_layers - 1):
            want = oracle.pack_layer(src_h, 0, wl.block_tables, wl.seq_lens, window=W)
            assert np.array_equal(to_host(packed[:nb // 2]), want), f"layer {layer} (W={W}) pack differs"
            oracle.unpack_layer(want, dst_before, 0, wl.dst_block_tables, wl.seq_lens, window=W)
            assert np.array_equal(to_host(dst[layer]), dst_before[0]), f"layer {layer} (W={W}) unpack differs"
            say(f"  layer {layer} W={W}: {nb} B bit-exact vs oracle")
    del src, dst, packed, again
    torch.cuda.empty_cache()


def _sparse(rng, lens, H, D, P, width):
    """A pool and tables `width` tokens wide of requests of these lengths."""
    need = [-(-int(n) // P) for n in lens]
    bt = np.full((len(lens), width // P), -1, dtype=np.int32)
    perm, at = rng.permutation(sum(need) + 3).astype(np.int32), 0
    for r, k in enumerate(need):
        bt[r, :k] = perm[at:at + k]
        at += k
    return bt, (1, sum(need) + 3, 2, P, H, D)


@pytest.mark.parametrize("R,W,P,P2", [(16, 1024, 16, 16), (17, 1024, 16, 16), (31, 500, 16, 48), (40, 500, 16, 16)])
def test_sparse_windows(tk, R, W, P, P2):
    """Windows of wide tables on both sides of 32 MiB of window capacity (1 KiB rows, two planes), over requests
    that are mostly shorter than the window."""
    H, D = 8, 64
    rng = np.random.default_rng(R + W)
    lens = np.array([[200, 0, 1, W - 1, W, W + 1, 37, 1500][r % 8] for r in range(R)], dtype=np.int32)
    (bt, shape), (bt2, shape2) = _sparse(rng, lens, H, D, P, 32768), _sparse(rng, lens, H, D, P2, 32768)
    src_h, dst_h = (rng.integers(0, 65536, size=s, dtype=np.uint16) for s in (shape, shape2))
    say(f"[window] sparse: {R} requests, window {W}, pages {P}->{P2}")
    want, want_dst = oracle.pack_layer(src_h, 0, bt, lens, window=W), dst_h.copy()
    oracle.unpack_layer(want, want_dst, 0, bt2, lens, window=W)
    src, dst, btd, bt2d, lensd = to_dev(src_h), to_dev(dst_h), to_dev(bt), to_dev(bt2), to_dev(lens)
    packed = to_dev(np.zeros(want.size + 16, np.uint16))
    tk.topkv_pack_layer_window(src, 0, R, btd, bt.shape[1], lensd, W, packed, dst_bytes=2 * want.size)
    tk.topkv_unpack_layer_window(packed, dst, 0, R, bt2d, bt2.shape[1], lensd, W, src_bytes=2 * want.size)
    torch.cuda.synchronize()
    got = to_host(packed)
    assert np.array_equal(got[:want.size], want) and not got[want.size:].any()
    assert np.array_equal(to_host(dst), want_dst)


@pytest.mark.parametrize("R", [24, 300])
def test_short_requests_in_windows(tk, R):
    """Requests of 200 tokens in windows of 1000 move in about the time that they take without a window, in
    tables as wide as they are (1.6 and 2.4 times it where the live tiles share few CUs)."""
    H, D, P, n = 8, 64, 16, 200
    rng = np.random.default_rng(R)
    bt, shape = _sparse(rng, [n] * R, H, D, P, 32768)
    src = torch.zeros(shape, dtype=torch.int16, device="cuda")
    packed = torch.zeros(2 * R * n * H * D, dtype=torch.int16, device="cuda")
    lens, wide = to_dev(np.full(R, n, np.int32)), to_dev(bt)
    exact = to_dev(np.ascontiguousarray(bt[:, :-(-n // P)]))
    say(f"[window] short requests: {R}")
    windowed = tk.prepare_pack_layer_window(src, 0, R, wide, wide.shape[1], lens, 1000, packed)
    plain = tk.prepare_pack_layer_window(src, 0, R, exact, exact.shape[1], lens, 0, packed)
    us = []
    for call in (windowed, plain) * 5:
        for _ in range(3):
            call()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(30):
            call()
        b.record()
        b.synchronize()
        us.append(a.elapsed_time(b) * 1000 / 30)
    windowed_us, plain_us = sorted(us[::2])[2], sorted(us[1::2])[2]
    say(f"[window] {R} requests of {n} tokens: window {windowed_us:.2f} us, plain {plain_us:.2f} us")
    assert windowed_us < 1.5 * plain_us + 1.0
