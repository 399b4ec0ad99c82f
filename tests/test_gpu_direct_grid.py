"""The layout-move direct and live grids at the sizes where they can go wrong, bit for bit against the
oracle: units of several page sizes, wave-uniform and per-lane spans, several granules, rows that are no
multiple of 16 bytes or shorter than that, windows, each tile size, packed regions too small, and block
tables much wider than their requests."""
import math
import sys

import numpy as np
import pytest
import torch

import oracle
import oracle.reshard as rs
from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu
WORDS = {1: np.uint8, 2: np.uint16, 4: np.uint32, 8: np.uint64}


@pytest.fixture(scope="module")
def tk():
    from paper_2607_28633_amd import topkv
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return topkv


def _tables(rng, lens, P):
    need = [-(-int(n) // P) for n in lens]
    NP = sum(need) + 3
    bt = np.full((len(lens), max([1] + need) + 1), -1, dtype=np.int32)
    perm, cur = rng.permutation(NP).astype(np.int32), 0
    for r, k in enumerate(need):
        bt[r, :k] = perm[cur:cur + k]
        cur += k
    return bt, NP


def _words(rng, n, eb):
    return rng.integers(0, 256, size=n * eb, dtype=np.uint8).view(WORDS[eb])


# heads, dim, elem, P, P2, lengths, head slice (first, count), shards, window
CASES = [
    # whole rows: per-lane units (72, 16, 22, 1.5 chunks a token) and wave-uniform ones, tile edges
    (1, 576, 2, 64, 16, [1, 63, 64, 65, 300], None, 1, 0),
    (1, 576, 2, 5, 7, [1, 34, 35, 36, 200], None, 1, 0),
    (1, 128, 2, 16, 1, [15, 16, 17, 511, 512, 513], None, 1, 0),
    (7, 25, 2, 16, 24, [23, 24, 25, 700], None, 1, 0),
    (3, 3, 2, 16, 9, [1, 2, 143, 145], None, 1, 0),          # 18-byte rows
    (1, 6, 1, 16, 4, [1, 2, 3, 63, 64, 65], None, 1, 0),     # 6-byte rows: short last runs
    (1, 5, 1, 3, 3, [1, 2, 7, 30], None, 1, 0),              # units shorter than a chunk: the general grid
    (8, 128, 2, 16, 64, [8192], None, 1, 0),                 # wave-uniform, one request: 8 chunks a lane
    (1, 129, 2, 16, 16, [40000, 1, 39999], None, 1, 0),      # per lane, 2 chunks: the longest grids
    (8, 128, 2, 16, 16, [2047, 2048, 2049], None, 1, 0),     # 8 chunks
    (8, 128, 2, 16, 16, [640, 1], None, 1, 0),               # 1 chunk
    # head slices and shards
    (8, 128, 2, 16, 16, [100, 1, 33], (2, 2), 1, 0),
    (8, 128, 2, 16, 64, [100, 1, 33], (0, 8), 4, 0),
    (6, 20, 2, 8, 16, [50, 9], (1, 4), 2, 0),                # 40-byte granules
    (6, 9, 1, 8, 16, [50, 9], (1, 4), 2, 0),                 # 18-byte granules
    # windows
    (8, 64, 2, 16, 16, [1, 127, 128, 129, 500, 0], None, 1, 128),
    (1, 576, 2, 64, 16, [1, 100, 101, 164, 500], None, 1, 100),
    (7, 25, 2, 16, 24, [23, 24, 300, 700], None, 1, 17),
    # windows of whole wave spans, 16 to 120 requests: 1, 1, 2 and 4 chunks per lane
    (1, 32, 2, 16, 16, [1023 + i for i in range(16)], None, 1, 1024),
    (1, 32, 2, 16, 16, [1000 + 3 * i for i in range(32)], None, 1, 1024),
    (1, 32, 2, 16, 16, [990 + 2 * i for i in range(64)], None, 1, 1024),
    (1, 32, 2, 16, 16, [i if i < 20 else 880 + i for i in range(120)], None, 1, 900),
    (1, 6, 1, 16, 4, [1, 9, 63, 64, 65], None, 1, 5),
    # several granules: 2 and 4 chunks per lane of whole spans, 2 of lanes with a unit each
    (8, 128, 2, 16, 64, [700, 650], (0, 8), 4, 0),
    (8, 128, 2, 16, 64, [1500, 1400], (0, 8), 4, 0),
    (6, 20, 2, 8, 16, [7000, 6990], (1, 4), 2, 0),
]


def _plan(H, hc, head, P, P2, kind, lens, S, W, width=None):
    """The host's plan for one move of a case: (whole wave spans, granules, chunks per lane or "live", workgroups)
    of the direct or live grid, None for the general one.  kind: pack, unpack, unpack_hm, pool or pool_hm."""
    hm = kind.endswith("hm")
    per = 1 if hm else hc // S
    gran, gpt = per * head, hc // per
    heads, scattered = gpt > 1, gpt > 1 or kind.startswith("pool")
    pages = [P] if kind == "pack" else [P2] if kind.startswith("unpack") else [P, P2]
    unit = 1 if heads or hc != H else math.gcd(*pages)
    if (gran if heads else unit * gran) < 16 or len(lens) > 1024:
        return None
    cpu = gpt * -(-gran // 16) if heads else -(-unit * gran // 16)
    tok = min((width or (max(1, -(-max(lens) // p)) + 1)) * p for p in pages)
    units = -(-tok // unit)
    if W:
        units = min(units, (W + unit - 2) // unit + 1)
    grid = lambda v: -(-units * cpu // (v * 256)) * 2 * len(lens)
    wave = cpu % 64 == 0
    v = 2 if not wave else 4 if scattered else 8
    while v > 1 and grid(v) < 512:
        v //= 2
    return (wave, heads, v if grid(v) <= 8192 else "live", grid(v))


def test_cases_reach_every_tile_size():
    """CASES together run every tile size of the direct grid that a batch can have, for each direction, whole
    spans and lanes, one granule and several."""
    seen = set()
    for H, D, eb, P, P2, lens, sl, S, W in CASES:
        for kind in ("pack", "unpack", "unpack_hm", "pool", "pool_hm"):
            p = _plan(H, (sl or (0, H))[1], D * eb, P, P2, kind, lens, 1 if kind.startswith("pool") else S, W)
            if p:
                seen.add((kind.split("_")[0],) + p[:3])
    want = {(way, wave, heads, v) for way in ("pack", "unpack", "pool") for wave in (False, True) for heads in (False, True)
            for v in ((1, 2) if not wave else (1, 2, 4) if heads or way == "pool" else (1, 2, 4, 8))}
    assert want <= seen, want - seen


@pytest.mark.parametrize("case", range(len(CASES)))
def test_direct_grid_parity(tk, case):
    H, D, eb, P, P2, lens, sl, S, W = CASES[case]
    C, (h0, hc) = 2, sl or (0, H)
    say(f"[direct_grid] case {case}: H{H} D{D} u{8 * eb} P{P}->{P2} lens {lens} heads {h0}+{hc} shards {S} window {W}")
    rng = np.random.default_rng(case)
    lens_h = np.array(lens, dtype=np.int32)
    (bt, NP), (bt2, NP2) = _tables(rng, lens, P), _tables(rng, lens, P2)
    src_h = _words(rng, NP * C * P * H * D, eb).reshape(1, NP, C, P, H, D)
    dst_h = _words(rng, NP2 * C * P2 * H * D, eb).reshape(1, NP2, C, P2, H, D)
    hm_h = _words(rng, NP2 * C * P2 * H * D, eb).reshape(1, NP2, C, H, P2, D)
    src, btd, bt2d, lensd, R = to_dev(src_h), to_dev(bt), to_dev(bt2), to_dev(lens_h), len(lens)
    cap = rs.packed_heads_elems(C, hc // S, D, lens, W)
    shard = dict(shards=S, shard_elems=cap)
    pool, to = rs.View(rs.POOL, src_h, 0, bt, h0), lambda kind, d: rs.View(kind, d, 0, bt2, h0)
    pv = tk.pool_view(src, 0, btd, bt.shape[1], h0)

    want = np.zeros(S * cap, WORDS[eb])
    rs.move_layer(pool, rs.View(rs.PACKED, want, **shard), lens_h, hc, W)
    packed = to_dev(np.zeros(S * cap + 16, WORDS[eb]))
    kv = tk.packed_view(packed, nbytes=cap * eb, shards=S)
    tk.topkv_move_layer(pv, kv, R, lensd, hc, W)
    torch.cuda.synchronize()
    got = to_host(packed)
    assert np.array_equal(got[:S * cap], want) and not got[S * cap:].any(), "pack"

    for kind, host in ((rs.POOL, dst_h), (rs.POOL_HEAD_MAJOR, hm_h)):
        dv = lambda d: tk.pool_view(d, 0, bt2d, bt2.shape[1], h0, kind == rs.POOL_HEAD_MAJOR)
        want_u, dst = host.copy(), to_dev(host)
        rs.move_layer(rs.View(rs.PACKED, want, **shard), to(kind, want_u), lens_h, hc, W)
        tk.topkv_move_layer(kv, dv(dst), R, lensd, hc, W)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(dst), want_u), f"unpack into {kind}"
        want_p, dst = host.copy(), to_dev(host)
        rs.move_layer(pool, to(kind, want_p), lens_h, hc, W)
        tk.topkv_move_layer(pv, dv(dst), R, lensd, hc, W)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(dst), want_p), f"pool to {kind}"


@pytest.mark.parametrize("H,D,eb,hc,S", [(8, 128, 2, 8, 1), (7, 25, 2, 7, 1), (8, 128, 2, 4, 2), (1, 6, 1, 1, 1)])
def test_direct_grid_short_regions(tk, H, D, eb, hc, S):
    """A packed side too small for the batch: whole pieces below each region's capacity move, nothing past it."""
    C, P, lens = 2, 16, [33, 5, 70]
    rng = np.random.default_rng(H + D)
    bt, NP = _tables(rng, lens, P)
    src_h = _words(rng, NP * C * P * H * D, eb).reshape(1, NP, C, P, H, D)
    full = rs.packed_heads_elems(C, hc // S, D, lens)
    whole = np.zeros(S * full, WORDS[eb])
    rs.move_layer(rs.View(rs.POOL, src_h, 0, bt, 0), rs.View(rs.PACKED, whole, shards=S, shard_elems=full),
                  np.array(lens, np.int32), hc)
    src, btd, lensd = to_dev(src_h), to_dev(bt), to_dev(np.array(lens, np.int32))
    piece = 16 // eb if (hc // S * D * eb) % 16 == 0 else 2 // eb  # elements of the widest aligned piece of a token
    for cap in (full - piece, full // 2 // piece * piece, 10 * piece):
        say(f"[direct_grid] short region H{H} D{D} u{8 * eb} shards {S}: {cap} of {full}")
        packed = to_dev(np.zeros(S * cap + 16, WORDS[eb]))
        kv = tk.packed_view(packed, nbytes=cap * eb, shards=S)
        tk.topkv_move_layer(tk.pool_view(src, 0, btd, bt.shape[1]), kv, 3, lensd, hc)
        torch.cuda.synchronize()
        got = to_host(packed)
        for s in range(S):
            assert np.array_equal(got[s * cap:(s + 1) * cap], whole[s * full:s * full + cap]), f"shard {s}"
        assert not got[S * cap:].any()
        back_h = _words(rng, src_h.size, eb).reshape(src_h.shape)
        back, want = to_dev(back_h), back_h.copy()
        tk.topkv_move_layer(kv, tk.pool_view(back, 0, btd, bt.shape[1]), 3, lensd, hc)
        torch.cuda.synchronize()
        marks, wide = np.zeros(S * full, WORDS[eb]), np.zeros(S * full, WORDS[eb])
        for s in range(S):
            marks[s * full:s * full + cap] = 1
            wide[s * full:s * full + cap] = whole[s * full:s * full + cap]
        moved, filled = np.zeros_like(back_h), back_h.copy()
        shard = dict(shards=S, shard_elems=full)
        rs.move_layer(rs.View(rs.PACKED, marks, **shard), rs.View(rs.POOL, moved, 0, bt, 0), np.array(lens, np.int32), hc)
        rs.move_layer(rs.View(rs.PACKED, wide, **shard), rs.View(rs.POOL, filled, 0, bt, 0), np.array(lens, np.int32), hc)
        assert np.array_equal(to_host(back), np.where(moved == 1, filled, want)), "unpack of a short region"


@pytest.mark.parametrize("H,D,eb,P,P2", [(2, 128, 2, 16, 1), (2, 128, 2, 1, 16), (1, 576, 1, 4, 1), (3, 1, 2, 16, 16),
                                         (1, 1, 1, 16, 8), (1, 2047, 1, 2, 2), (1, 2048, 1, 2, 2)])
@pytest.mark.parametrize("short", [False, True])
def test_small_planes(tk, H, D, eb, P, P2, short):
    """Page planes below 4 KiB (and one at it) through pack, unpack and the layer engine, with a packed
    buffer that holds the batch or ends inside the last request, which then does not move at all."""
    C, L, lens = 2, 3, [1, 0, 40, 515]
    rng = np.random.default_rng(H + D + P)
    (bt, NP), (bt2, NP2) = _tables(rng, lens, P), _tables(rng, lens, P2)
    src_h = _words(rng, L * NP * C * P * H * D, eb).reshape(L, NP, C, P, H, D)
    dst_h = _words(rng, L * NP2 * C * P2 * H * D, eb).reshape(L, NP2, C, P2, H, D)
    n = C * H * D * sum(lens)
    kept = n - C * H * D * lens[-1] if short else n               # elements that move
    cap = (n - 1) * eb if short else n * eb
    say(f"[small_planes] H{H} D{D} u{8 * eb} P{P}->{P2} short {short}")
    src, btd, bt2d, lensd = to_dev(src_h), to_dev(bt), to_dev(bt2), to_dev(np.array(lens, np.int32))
    used = lens[:-1] + [0] if short else lens
    packs = [oracle.pack_layer(src_h, l, bt, np.array(used, np.int32)) for l in range(L)]
    want_dst = dst_h.copy()
    for l in range(L):
        oracle.unpack_layer(packs[l], want_dst, l, bt2, np.array(used, np.int32))

    stride = n + 5
    packed, dst = to_dev(np.zeros(L * stride, WORDS[eb])), to_dev(dst_h)
    for l in range(L):
        part = packed[l * stride:(l + 1) * stride]
        tk.topkv_pack_layer_batched(src, l, len(lens), btd, bt.shape[1], lensd, part, dst_bytes=cap)
        tk.topkv_unpack_layer_batched(part, dst, l, len(lens), bt2d, bt2.shape[1], lensd, src_bytes=cap)
    torch.cuda.synchronize()
    got = to_host(packed).reshape(L, stride)
    assert all(np.array_equal(got[l][:kept], packs[l]) and not got[l][kept:].any() for l in range(L))
    assert np.array_equal(to_host(dst), want_dst)

    # the engine: a layer stride one element short of the batch, or a range whose last layer's block is
    layer = (n - 1) if short else n
    packed, dst = to_dev(np.zeros(L * n + 16, WORDS[eb])), to_dev(dst_h)
    tk.topkv_engine_pack_layers(src, 0, L, len(lens), btd, bt.shape[1], lensd, packed, layer * eb,
                                packed_bytes=((L - 1) * layer + n - (0 if short else 1)) * eb)
    tk.topkv_engine_unpack_layers(packed, layer * eb, dst, 0, L, len(lens), bt2d, bt2.shape[1], lensd,
                                  packed_bytes=((L - 1) * layer + n - (0 if short else 1)) * eb)
    torch.cuda.synchronize()
    got, want_dst = to_host(packed), dst_h.copy()
    for l in range(L):
        whole = not short and l < L - 1
        part = packs[l] if short or whole else packs[l][:C * H * D * sum(lens[:-1])]
        assert np.array_equal(got[l * layer:l * layer + part.size], part), f"engine layer {l}"
        oracle.unpack_layer(part, want_dst, l, bt2, np.array(used if short or whole else lens[:-1] + [0], np.int32))
    assert np.array_equal(to_host(dst), want_dst)


# 64-byte rows in 16-token pages (one wave span a page plane): each tile size of the one-request grid
ROWS = [1, 15, 16, 17, 1024, 1025, 8192, 8193, 16385, 24577, 32769, 49153, 65537, 98305, 200001, 300000]


@pytest.mark.parametrize("n", ROWS)
def test_one_request_rows(tk, n):
    H, D, P, P2, C = 1, 32, 16, 32, 2
    say(f"[direct_grid] one request of {n} tokens")
    rng = np.random.default_rng(n)
    lens = np.array([n], dtype=np.int32)
    (bt, NP), (bt2, NP2) = _tables(rng, lens, P), _tables(rng, lens, P2)
    bt[0, (n // P) // 2] = NP + 7 if n > 1024 else bt[0, (n // P) // 2]      # a page outside the pool
    src_h = _words(rng, 2 * NP * C * P * H * D, 2).reshape(2, NP, C, P, H, D)
    dst_h = _words(rng, 2 * NP2 * C * P2 * H * D, 2).reshape(2, NP2, C, P2, H, D)
    t = np.arange(n)
    page = bt[0][t // P]
    there = page < NP
    want = np.zeros((C, n, H, D), dtype=np.uint16)
    want[:, there] = src_h[1][page[there], :, t[there] % P].transpose(1, 0, 2, 3)
    want_u = dst_h.copy()
    full = _words(rng, C * n * H * D, 2).reshape(C, n, H, D)
    want_u[1][bt2[0][t // P2], :, t % P2] = full.transpose(1, 0, 2, 3)
    src, btd, bt2d, lensd = to_dev(src_h), to_dev(bt), to_dev(bt2), to_dev(lens)
    size = C * n * H * D
    wide = torch.full((1, bt.shape[1] * 3), -1, dtype=torch.int32, device="cuda")
    wide[:, :bt.shape[1]] = btd
    for table, host_len in ((btd, True), (btd, False), (wide, False)):
        packed = torch.zeros(size + 8, dtype=torch.int16, device="cuda")
        dst, body = to_dev(dst_h), to_dev(full.reshape(-1))
        if host_len:
            tk.topkv_pack_layer(src, 1, table, n, packed)
            tk.topkv_unpack_layer(body, dst, 1, bt2d, n)
        else:
            tk.topkv_pack_layer_batched(src, 1, 1, table, table.shape[1], lensd, packed, 2 * size)
            tk.topkv_unpack_layer_batched(body, dst, 1, 1, bt2d, bt2d.shape[1], lensd)
        torch.cuda.synchronize()
        got = to_host(packed).view(np.uint16)
        assert np.array_equal(got[:size].reshape(want.shape), want) and not got[size:].any(), "pack"
        assert np.array_equal(to_host(dst), want_u), "unpack"
    packed, dst = torch.zeros(size, dtype=torch.int16, device="cuda"), to_dev(dst_h)
    tk.topkv_pack_layer_batched(src, 1, 1, btd, bt.shape[1], lensd, packed, 2 * size - 2)
    tk.topkv_unpack_layer_batched(body, dst, 1, 1, bt2d, bt2d.shape[1], lensd, 2 * size - 2)
    torch.cuda.synchronize()
    assert not to_host(packed).any() and np.array_equal(to_host(dst), dst_h), "a request that does not fit moved"



# one request on both sides of the page grid's share (planes of 8 KiB, 8 MiB of layer) and of the rows grid's
# change from 64 to 24 and 32 KiB tiles (16 MiB, 18 MiB and more)
@pytest.mark.parametrize("H,D,n", [(2, 128, 40), (2, 128, 8192), (2, 128, 8193), (1, 128, 16384), (1, 129, 16384),
                                   (8, 128, 4096), (8, 128, 4097), (8, 128, 4600), (8, 128, 4700)])
def test_one_request_layer(tk, H, D, n):
    P, P2, C = 16, 32, 2
    say(f"[direct_grid] one request of {n} tokens, {H} heads of {D}")
    rng = np.random.default_rng(n + H)
    lens = np.array([n], dtype=np.int32)
    (bt, NP), (bt2, NP2) = _tables(rng, lens, P), _tables(rng, lens, P2)
    src_h, dst_h = _words(rng, NP * C * P * H * D, 2).reshape(1, NP, C, P, H, D), _words(rng, NP2 * C * P2 * H * D, 2).reshape(1, NP2, C, P2, H, D)
    want, want_dst = oracle.pack_layer(src_h, 0, bt, lens), dst_h.copy()
    oracle.unpack_layer(want, want_dst, 0, bt2, lens)
    need = -(-n // P)
    src, lensd, exact, exact2 = to_dev(src_h), to_dev(lens), to_dev(bt[:, :need].copy()), to_dev(bt2[:, :-(-n // P2)].copy())
    for host_len in (False, True):
        packed, dst = to_dev(np.zeros(want.size + 8, np.uint16)), to_dev(dst_h)
        if host_len:
            tk.topkv_pack_layer(src, 0, exact, n, packed)
            tk.topkv_unpack_layer(packed, dst, 0, exact2, n)
        else:
            tk.topkv_pack_layer_batched(src, 0, 1, exact, exact.shape[1], lensd, packed, 2 * want.size)
            tk.topkv_unpack_layer_batched(packed, dst, 0, 1, exact2, exact2.shape[1], lensd, 2 * want.size)
        torch.cuda.synchronize()
        got = to_host(packed)
        assert np.array_equal(got[:want.size], want) and not got[want.size:].any(), "pack"
        assert np.array_equal(to_host(dst), want_dst), "unpack"


DIRECT_SLOTS = 8192                                          # most workgroups of a direct grid of device lengths
# windows whose grid is longer than that although most requests are short
WIDE_WINDOWS = [(1, 576, 2, 64, 16, [2, 0, 3100, 150, 64, 65] * 10, None, 1, 3000),
                (7, 25, 2, 16, 24, [9, 2300, 0, 1, 8, 33] * 10, None, 1, 2000),
                (8, 128, 2, 16, 64, [9, 300, 0, 1, 8, 33] * 10, (2, 2), 1, 2000)]


def _wide(row, R, C):
    """Tokens of a table whose direct grid is past DIRECT_SLOTS in its largest (2048-chunk) tiles."""
    return -(-(DIRECT_SLOTS + 1) // (R * C)) * 2048 * 16 // row + 2048


@pytest.mark.parametrize("case", [i for i, c in enumerate(CASES) if not c[8]] + [len(CASES) + i for i in range(len(WIDE_WINDOWS))])
def test_wide_tables(tk, case, monkeypatch):
    """Every kind of move with block tables much wider than the requests (entries past them hold anything):
    the live grid."""
    H, D, eb, P, P2, lens, sl, S, W = (CASES + WIDE_WINDOWS)[case]
    hc, narrow, R = (sl or (0, H))[1], _tables, len(lens)
    wide = 0 if W else min(_wide(hc * D * eb, R, 2), (1 << 31) // (R * 2 * hc * D * eb) - 64)

    def tables(rng, lens, page):
        bt, NP = narrow(rng, lens, page)
        out = rng.integers(-(1 << 31), 1 << 31, size=(R, max(bt.shape[1], wide // page)), dtype=np.int64).astype(np.int32)
        out[:, :bt.shape[1]] = np.where(bt < 0, out[:, :bt.shape[1]], bt)
        return out, NP
    monkeypatch.setattr(sys.modules[__name__], "_tables", tables)
    monkeypatch.setattr(sys.modules[__name__], "CASES", CASES + WIDE_WINDOWS)
    test_direct_grid_parity(tk, case)


@pytest.mark.parametrize("short", [False, True])
def test_small_planes_in_wide_tables(tk, short, monkeypatch):
    """Plain layers and the layer engine over small page planes, with tables that put them in the live grid."""
    narrow = _tables

    def tables(rng, lens, page):
        bt, NP = narrow(rng, lens, page)
        return np.concatenate([bt, np.full((len(lens), 40000 // page), -1, np.int32)], axis=1), NP
    monkeypatch.setattr(sys.modules[__name__], "_tables", tables)
    test_small_planes(tk, 2, 128, 2, 16, 1, short)
    test_small_planes(tk, 2, 128, 2, 1, 16, short)


@pytest.mark.parametrize("head_major", [False, True])
@pytest.mark.parametrize("full", [False, True])
def test_large_moves_between_pools(tk, full, head_major):
    """Moves between pools past 32 tiles of 4 chunks per compute unit take tiles of 8: as many workgroups as
    the destination pool holds tiles (short requests, most of them with nothing to do), or 24 per compute
    unit that go on to further tiles (requests that fill the pool)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    H, D, C, P, P2, R = 8, 128, 2, 16, 64, 45
    tile = 4 * 256 * 16 // (H * D * 2)                          # tokens of one plane in 4 chunks a lane
    most = 32 * cus * tile // C                                 # tokens of as many tiles
    rng = np.random.default_rng(17 + full)
    lens = [(most * 2 // R & ~63) + int(k) for k in rng.integers(1, 64, size=R)] if full else \
        [int(k) for k in rng.choice([0, 1, 15, 16, 17, 63, 64, 65, 130], size=R)]
    width = max(lens) if full else 2 * most // R
    pools = []
    for page in (P, P2):
        need = [-(-n // page) for n in lens]
        NP = max(sum(need) + 3, most * 5 // 4 // page)
        bt = np.full((R, -(-width // page) + 1), NP, dtype=np.int32)      # entries past a request: outside the pool
        perm, at = rng.permutation(NP).astype(np.int32), 0
        for r, k in enumerate(need):
            bt[r, :k] = perm[at:at + k]
            at += k
        pools.append((bt, NP, to_dev(bt)))
    (bt, NP, bt_d), (bt2, NP2, bt2_d) = pools
    src = torch.randint(-32768, 32768, (1, NP, C, P, H, D), dtype=torch.int16, device="cuda")
    dst = torch.full((1, NP2, C, H, P2, D) if head_major else (1, NP2, C, P2, H, D), 0x5A5A, dtype=torch.int16, device="cuda")
    want = dst.clone()
    rows = want[0].transpose(2, 3) if head_major else want[0]            # [page, plane, slot, head, dim]
    for r, n in enumerate(lens):
        t = torch.arange(n, device="cuda")
        rows[bt2_d[r].long()[t // P2], :, t % P2] = src[0, bt_d[r].long()[t // P], :, t % P]
    say(f"[direct] between pools: {sum(lens)} tokens of {R} requests, pool of {NP2 * P2}, head-major {head_major}")
    tk.prepare_move_layer(tk.pool_view(src, 0, bt_d, bt.shape[1]),
                          tk.pool_view(dst, 0, bt2_d, bt2.shape[1], head_major=head_major),
                          R, to_dev(np.array(lens, dtype=np.int32)), H)()
    torch.cuda.synchronize()
    assert torch.equal(dst, want)


def _us(call, n=30):
    for _ in range(3):
        call()
    best = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        b.synchronize()
        best.append(a.elapsed_time(b) * 1000 / n)
    return sorted(best)[2]


@pytest.mark.parametrize("kind", ["slice", "reblock", "tokens"])
def test_table_width_costs_little(tk, kind):
    """64 requests of 100 tokens in tables of 131072 tokens: the launch follows the lengths (about 2 times
    the exact tables' launch), where a grid over the tables' entries takes 40 to 100 times it."""
    R, n, C = 64, 100, 2
    H, D, P, P2 = {"slice": (8, 128, 16, 16), "reblock": (1, 576, 64, 16), "tokens": (2, 128, 16, 1)}[kind]
    rng = np.random.default_rng(1)
    (bt, NP), (bt2, NP2) = _tables(rng, [n] * R, P), _tables(rng, [n] * R, P2)
    src = torch.zeros((1, NP, C, P, H, D), dtype=torch.int16, device="cuda")
    dst = torch.zeros((1, NP2, C, P2, H, D), dtype=torch.int16, device="cuda")
    packed = torch.zeros(C * R * n * H * D, dtype=torch.int16, device="cuda")
    lens = to_dev(np.full(R, n, np.int32))
    us = {}
    for width in (n, 131072):
        t, t2 = (to_dev(np.pad(b, ((0, 0), (0, max(0, width // p - b.shape[1]))), constant_values=-1)) for b, p in ((bt, P), (bt2, P2)))
        say(f"[direct_grid] {kind}: tables {tuple(t.shape)} and {tuple(t2.shape)}")
        if kind == "slice":
            call = tk.prepare_pack_layer_heads(src, 0, R, t, t.shape[1], lens, 2, 2, packed)
        elif kind == "reblock":
            call = tk.prepare_move_layer(tk.pool_view(src, 0, t, t.shape[1]), tk.pool_view(dst, 0, t2, t2.shape[1]), R, lens, H)
        else:
            call = tk.prepare_unpack_layer_window(packed, dst, 0, R, t2, t2.shape[1], lens, 0)
        us[width] = _us(call)
        torch.cuda.synchronize()
    say(f"[direct_grid] {kind}: {us}")
    assert us[131072] < 8 * us[n]
