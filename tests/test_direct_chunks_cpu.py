"""CPU model of the index arithmetic of the layout-move direct grid (kv_reshard_direct_kernel of
csrc/reshard.hip and the host's plan for it), of the live grid's tiles and of the one-request rows grid: units, 16-byte chunks, a run's last
chunk moved back to end with the run, runs that are short or cut by the packed capacity
byte by byte, windows, packed capacities and shard regions.  Every access is
checked against its buffer, and the bytes that arrive against the oracle's
definition of the move (and, where a capacity cuts the packed side short,
against the piece-wise rule of the general path).  Chunks of a run may repeat
bytes: the model checks that repeated writes carry the same values."""
import math
import random

import numpy as np
import pytest

import oracle
import oracle.reshard as rs

NT = 256


def make_div(d):
    s = 0
    while (1 << s) < d:
        s += 1
    return d, ((((1 << 32) * ((1 << s) - d)) // d) + 1) & 0xFFFFFFFF, s


def fdiv(n, f):
    n = np.asarray(n, dtype=np.uint64)
    assert (n < (1 << 31)).all()
    return ((((n * np.uint64(f[1])) >> np.uint64(32)) + n) >> np.uint64(f[2])).astype(np.int64)


class Side:
    """A pool (slot-major or head-major) or a packed buffer, as flat bytes."""

    def __init__(self, kind, data, layer=0, tables=None, head0=0):
        self.kind, self.data, self.layer, self.tables, self.head0 = kind, data, layer, tables, head0
        self.flat = data.view(np.uint8).reshape(-1)
        if kind == rs.PACKED:
            return
        L, self.NP, self.C = data.shape[:3]
        eb, self.D = data.dtype.itemsize, data.shape[5]
        self.P, self.H = (data.shape[3], data.shape[4]) if kind == rs.POOL else (data.shape[4], data.shape[3])
        head = self.D * eb
        self.row, self.plane = self.H * head, self.H * head * self.P
        self.page = self.plane * self.C
        self.base = layer * self.NP * self.page
        self.head_bytes = head * self.P if kind == rs.POOL_HEAD_MAJOR else head
        self.slot = head if kind == rs.POOL_HEAD_MAJOR else self.row


def model_move(src, dst, lens, hc, window, cap, shards, vb, vpt, strict=False):
    """Runs the grid; returns whether the host takes it, dst.flat modified."""
    geo = src if src.kind != rs.PACKED else dst
    head = geo.D * geo.data.dtype.itemsize
    pools = [s for s in (src, dst) if s.kind != rs.PACKED]
    per_gran = hc // shards if all(s.kind != rs.POOL_HEAD_MAJOR for s in pools) else 1
    gran, gpt = per_gran * head, hc // per_gran
    heads = gpt > 1
    unit = 0
    for s in pools:
        if heads or hc != s.H:
            unit = 1
            break
        unit = math.gcd(unit, s.P)
    cpg = (gran + 15) // 16
    cpu = gpt * cpg if heads else (unit * gran + 15) // 16
    if (gran if heads else unit * gran) < 16 or (src.kind == rs.PACKED and cap < 16):
        return False
    max_tok = min(s.tables.shape[1] * s.P for s in pools)
    max_units = -(-max_tok // unit)
    grid_units = max_units
    if window > 0:
        grid_units = min(max_units, (window + unit - 2) // unit + 1)
    tiles = -(-grid_units * cpu // (vpt * NT))
    d_unit, d_cpu, d_cpg, d_gps = make_div(unit), make_div(cpu), make_div(cpg), make_div(gpt // shards)
    written = {}
    before = 0
    for r in range(len(lens)):
        n = min(max(int(lens[r]), 0), max_tok)
        start = n - window if 0 < window < n else 0
        kept = n - start
        unit0 = int(fdiv(start, d_unit)) if window > 0 else 0
        end = (int(fdiv(n - 1, d_unit)) + 1 - unit0) * cpu if n > 0 else 0
        assert end <= grid_units * cpu, "the grid covers the request"
        for c in range(geo.C):
            if strict and geo.C * (before + kept) * (gpt // shards) * gran > cap:
                continue
            idx = np.arange(min(tiles * vpt * NT, end + 3 * NT))   # tiles past the end exit
            idx = idx[(idx // (vpt * NT)) * (vpt * NT) < end]
            if not idx.size:
                continue
            live = idx < end
            rel = np.where(live, fdiv(idx, d_cpu), 0)
            m = idx - rel * cpu
            u = unit0 + rel
            first = u * unit
            last = np.minimum(first + unit, n)
            t = np.maximum(first, start)
            k = fdiv(m, d_cpg) if heads else np.zeros_like(m)
            at = (m - k * cpg if heads else m) * 16
            run = np.full_like(m, gran) if heads else (last - t) * gran
            tok = geo.C * before + c * kept + (t - start)
            sh = fdiv(k, d_gps) if heads else np.zeros_like(k)
            off = (tok * d_gps[0] + (k - sh * d_gps[0])) * gran if heads else tok * gran
            region = (gpt // shards if heads else 1) * gran
            cut = (geo.C * before + c * kept + kept) * region > cap
            fit = np.where(off + run > cap, np.where(off < cap, (cap - off) & -vb, 0), run)
            vec = live & (run >= 16) & (not cut)                   # a run's chunks move as vectors
            b = np.where(vec, np.minimum(at, run - 16), at)
            size = np.where(vec & (at < run), 16, np.where(live & ~vec & (at < fit), np.minimum(fit - at, 16), 0))
            packed = sh * cap + off
            place, ok, loads = [], np.ones(len(m), bool), None
            for s in (src, dst):
                if s.kind == rs.PACKED:
                    place.append(packed)
                    continue
                i = fdiv(u, make_div(s.P // unit))
                assert (i >= 0).all() and (i < s.tables.shape[1]).all(), "table index"
                page = s.tables[r][i].astype(np.int64)
                inside = (page >= 0) & (page < s.NP)
                ok &= inside
                place.append(s.base + page * s.page + c * s.plane + (t - i * s.P) * s.slot + s.head0 * s.head_bytes +
                             k * (per_gran * s.head_bytes))
                if s is src:
                    loads = inside
            # every lane loads 16 bytes: of its run, or from the source's start
            usable = vec & (loads if loads is not None else True)
            voff = np.where(run >= 16, np.minimum(at, run - 16), 0)
            base = 0 if src.kind == rs.PACKED else src.base
            lo = np.where(usable, place[0] + voff, base + (voff if src.kind != rs.PACKED else 0))
            assert (lo >= 0).all() and (lo + 16 <= src.flat.size).all(), "load"
            if src.kind == rs.PACKED:
                assert (lo[usable] + 16 <= (sh * cap)[usable] + cap).all(), "load within the region"
            for j in np.nonzero(ok & (size > 0))[0]:
                z, x0, o = int(size[j]), int(place[0][j] + b[j]), int(place[1][j] + b[j])
                assert 0 <= x0 and x0 + z <= src.flat.size, "source access"
                assert 0 <= o and o + z <= dst.flat.size, "destination access"
                for x in range(z):
                    v = src.flat[x0 + x]
                    assert written.setdefault(o + x, v) == v, "two values for one byte"
        before += kept
    for o, v in written.items():
        dst.flat[o] = v
    return True


def _case(seed, capped=False):
    rng = random.Random(seed)
    npr = np.random.default_rng(seed)
    C, H, D, eb = rng.choice([1, 2]), rng.randint(1, 6), rng.choice([1, 2, 5, 8, 16, rng.randint(1, 40)]), rng.choice([1, 2, 4])
    dt = {1: np.uint8, 2: np.uint16, 4: np.uint32}[eb]
    lens = np.array([rng.choice([0, 1, rng.randint(1, 70)]) for _ in range(rng.randint(1, 4))], dtype=np.int32)
    kinds = rng.choice([("pool", "packed"), ("packed", "pool"), ("pool", "packed"), ("packed", "pool"), ("pool", "pool"),
                        ("pool", "hm"), ("hm", "packed"), ("packed", "hm")])
    hc = rng.choice([H, H, rng.randint(1, H)])
    window = rng.choice([0, 0, rng.randint(1, 50)])
    shards = rng.choice([d for d in range(1, hc + 1) if hc % d == 0]) if "packed" in kinds else 1
    kept = sum(min(int(n), window) if window else int(n) for n in lens)
    elems = C * (hc // shards) * D * kept
    cap = elems + rng.choice([0, 0, 5])
    if capped and elems:
        cap = rng.randint(1, elems)
    sides = []
    for which, kind in enumerate(kinds):
        if kind == "packed":
            data = npr.integers(0, 255, size=max(1, shards * cap) * eb, dtype=np.uint8).view(dt)
            sides.append((rs.PACKED, data, 0, None, 0))
            continue
        P = rng.choice([1, 2, 4, 8, 16, rng.randint(1, 24)])
        need = [-(-int(n) // P) for n in lens]
        NP = sum(need) + rng.randint(1, 3)
        bt = np.full((len(lens), max([1] + need) + rng.randint(0, 2)), -1, dtype=np.int32)
        perm, cur = npr.permutation(NP).astype(np.int32), 0
        for r, q in enumerate(need):
            bt[r, :q] = perm[cur:cur + q]
            cur += q
        shape = (2, NP, C, H, P, D) if kind == "hm" else (2, NP, C, P, H, D)
        data = npr.integers(0, 255, size=int(np.prod(shape)) * eb, dtype=np.uint8).view(dt).reshape(shape)
        sides.append((rs.POOL if kind == "pool" else rs.POOL_HEAD_MAJOR, data, rng.randint(0, 1), bt, rng.randint(0, H - hc)))
    return dict(lens=lens, hc=hc, window=window, shards=shards, cap=cap, eb=eb, D=D, C=C, sides=sides, vpt=rng.choice([1, 2, 4, 8]))


@pytest.mark.parametrize("chunk", range(8))
def test_chunks_match_the_oracle(chunk):
    taken = 0
    for seed in range(100 * chunk, 100 * chunk + 100):
        c = _case(seed)
        s, d = c["sides"]
        if not c["lens"].any():
            continue
        out = d[1].copy()
        if not model_move(Side(*s), Side(d[0], out, *d[2:]), c["lens"], c["hc"], c["window"], c["cap"] * c["eb"]
                          if rs.PACKED in (s[0], d[0]) else (1 << 62), c["shards"], c["eb"], c["vpt"]):
            continue
        taken += 1
        want = d[1].copy()
        shard = dict(shards=c["shards"], shard_elems=c["cap"])
        rs.move_layer(rs.View(*s, **(shard if s[0] == rs.PACKED else {})),
                      rs.View(d[0], want, *d[2:], **(shard if d[0] == rs.PACKED else {})), c["lens"], c["hc"], c["window"])
        assert np.array_equal(out, want), f"seed {seed}"
    assert taken >= 30


@pytest.mark.parametrize("chunk", range(4))
def test_capacity_cuts_at_the_general_paths_piece(chunk):
    """A packed side (or shard region) too small for the batch: exactly the
    whole vb-byte pieces below its capacity move, as in the general path; with
    `strict`, whole requests."""
    for seed in range(5000 + 60 * chunk, 5060 + 60 * chunk):
        c = _case(seed, capped=True)
        s, d = c["sides"]
        if rs.PACKED not in (s[0], d[0]) or not c["lens"].any():
            continue
        cap, S, eb = c["cap"], c["shards"], c["eb"]
        vb = eb                                                    # a piece width the general path may take
        out = d[1].copy()
        if not model_move(Side(*s), Side(d[0], out, *d[2:]), c["lens"], c["hc"], c["window"], cap * eb, S, vb, c["vpt"]):
            continue
        # the same move with room for everything, then only elements below each region's capacity
        kept = sum(min(int(n), c["window"]) if c["window"] else int(n) for n in c["lens"])
        full = c["C"] * (c["hc"] // S) * c["D"] * kept
        def widen(data):
            wide = np.zeros(S * full, data.dtype)
            for x in range(S):
                wide[x * full:x * full + cap] = data[x * cap:(x + 1) * cap]
            return wide
        shard = dict(shards=S, shard_elems=full)
        if d[0] == rs.PACKED:
            wide = widen(d[1])
            rs.move_layer(rs.View(*s), rs.View(d[0], wide, **shard), c["lens"], c["hc"], c["window"])
            want = np.concatenate([wide[x * full:x * full + cap] for x in range(S)])
        else:
            a, b = d[1].copy(), d[1].copy()
            marks = widen(np.zeros(S * cap, d[1].dtype))
            for x in range(S):
                marks[x * full:x * full + cap] = 1
            ones = d[1].copy()
            ones[...] = 0
            rs.move_layer(rs.View(rs.PACKED, marks, **shard), rs.View(d[0], ones, *d[2:]), c["lens"], c["hc"], c["window"])
            rs.move_layer(rs.View(rs.PACKED, widen(s[1]), **shard), rs.View(d[0], a, *d[2:]), c["lens"], c["hc"], c["window"])
            want = np.where(ones == 1, a, b)
        assert np.array_equal(out, want), f"seed {seed}"


def test_strict_moves_whole_requests():
    rng = np.random.default_rng(3)
    pool = rng.integers(0, 255, size=(1, 12, 2, 4, 3, 5), dtype=np.uint8)
    bt = rng.permutation(12).reshape(3, 4).astype(np.int32)
    lens, row = np.array([7, 9, 3], np.int32), 15
    want = oracle.pack_layer(pool, 0, bt, lens)
    for cap in (2 * row * 19, 2 * row * 19 - 1, 2 * row * 16, 2 * row * 16 - 1, 2 * row * 7 - 1):
        out = np.full(2 * row * 19, 7, np.uint8)
        assert model_move(Side(rs.POOL, pool, 0, bt), Side(rs.PACKED, out), lens, 3, 0, cap, 1, 1, 1, strict=True)
        whole = max([0] + [2 * row * x for x in (7, 16, 19) if 2 * row * x <= cap])
        assert np.array_equal(out[:whole], want[:whole]) and (out[whole:] == 7).all()


def _live_tiles(lens, planes, unit, cpu, window, max_tok, tile):
    """live_prefix: each request's live tiles over all planes and kept tokens, as exclusive prefix sums."""
    d_unit, first, kept, clamped = make_div(unit), [0], [0], []
    for n in lens:
        n = min(max(int(n), 0), max_tok)
        clamped.append(n)
        start = n - window if 0 < window < n else 0
        units = int(fdiv(n - 1, d_unit)) + 1 - int(fdiv(start, d_unit)) if n > 0 else 0
        first.append(first[-1] + planes * -(-units * cpu // tile))
        kept.append(kept[-1] + n - start)
    return first, kept[:-1], clamped


def _tile_owner(first, R, t):
    """tile_owner: two rounds of 64 lanes' votes."""
    step = (R + 63) >> 6
    group = (sum(lane * step < R and first[lane * step if lane * step < R else 0] <= t for lane in range(64)) - 1) * step
    if step == 1:
        return group
    return group + sum(lane < step and group + lane < R and first[group + lane] <= t for lane in range(64)) - 1


@pytest.mark.parametrize("R", [1, 2, 63, 64, 65, 127, 128, 129, 200, 1000, 1024])
def test_live_grid_visits_every_tile_once(R):
    """The grid that follows the lengths: its tile indices name every (request, plane, tile) with tokens
    once, with the packed offset of the direct grid's sum, whatever requests are empty."""
    rng = random.Random(R)
    for trial in range(6):
        planes, unit, cpu, tile = rng.choice([1, 2, 3]), rng.choice([1, 7, 16, 64]), rng.choice([1, 22, 64, 72]), 256 * rng.choice([2, 4, 8])
        window, max_tok = rng.choice([0, 0, 100]), 3000
        share = [0.0, 0.1, 0.9, 1.0][trial % 4]                     # of empty or negative lengths
        lens = [rng.choice([0, -1]) if rng.random() < share else rng.choice([1, rng.randint(1, 300), 4000]) for _ in range(R)]
        if trial == 5:
            lens = [0] * (R - 1) + [17]
        first, kept, clamped = _live_tiles(lens, planes, unit, cpu, window, max_tok, tile)
        want = []
        for r, n in enumerate(clamped):
            start = n - window if 0 < window < n else 0
            end = ((n - 1) // unit + 1 - start // unit) * cpu if n else 0
            want += [(r, c, x) for c in range(planes) for x in range(-(-end // tile))]
            assert kept[r] == sum(min(k, window) if window else k for k in clamped[:r])
        got = []
        for t in range(first[R]):
            r = _tile_owner(first, R, t)
            tiles = (first[r + 1] - first[r]) // planes
            local = t - first[r]
            got.append((r, local // tiles, local % tiles))
        assert got == want


@pytest.mark.parametrize("pack", [True, False])
def test_rows_grid(pack):
    """kv_rows_kernel: every early table lookup inside the row, every load inside its buffer, and the chunks that
    arrive: one request's plane as one run of 16-byte chunks, pages outside the pool and chunks past the tokens left."""
    rng = random.Random(11 + pack)
    for trial in range(60):
        per_token, planes = rng.choice([4, 16, 64, 72, 128]), rng.choice([1, 2])
        P = 64 // math.gcd(64, per_token) * rng.choice([1, 2, 4])   # tokens a page: page planes of whole wave spans
        per_page, vpt = P * per_token, rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        n = rng.choice([0, 1, P, P + 1, rng.randint(1, 60)])
        stride = max(1, -(-n // P)) + rng.choice([0, 0, 3])
        pages = -(-n // P) + 2
        table = [rng.choice([-1, pages + 5]) if rng.random() < 0.2 else x for x in rng.sample(range(pages), -(-n // P))]
        table += [rng.choice([-7, 1 << 30]) for _ in range(stride - len(table))]
        tok_cap, fits = stride * P, rng.random() < 0.9
        total = min(max(n, 0), tok_cap) * per_token
        max_total = total + rng.choice([0, 5]) if fits else total - 1
        div = make_div(per_page)
        pool_chunks, moved = pages * planes * per_page, {}
        grid = -(-(tok_cap * per_token) // (vpt * NT))
        for block in range(grid):
            for c in range(planes):
                for wave in range(4):
                    base = block * NT * vpt + wave * 64
                    look = fdiv(np.array([base + min(lane, vpt - 1) * NT for lane in range(64)]), div)
                    look = np.minimum(look, stride - 1)
                    assert (look >= 0).all() and (look < stride).all()
                    if base >= total or total > max_total:
                        continue
                    for j in range(vpt):
                        first, entry = base + j * NT, table[look[j]]
                        usable = first < total and 0 <= entry < pages
                        m = first - int(fdiv(first, div)) * per_page
                        for lane in (0, 1, 63):
                            at = c * per_page + (entry * planes * per_page + m if usable else 0) + lane
                            load = at if pack else c * total + min(first + lane, total - 1)
                            assert 0 <= load < (pool_chunks if pack else planes * total)
                            if usable and first + lane < total:
                                there, here = (at, c * total + first + lane)
                                assert 0 <= there < pool_chunks and here < planes * total
                                assert moved.setdefault(here, there) == there
        want = {}
        if total <= max_total:
            for c in range(planes):
                for q in range(total):
                    if q % 64 in (0, 1, 63) and 0 <= table[q // per_page] < pages:
                        want[c * total + q] = (table[q // per_page] * planes + c) * per_page + q % per_page
        assert moved == want
