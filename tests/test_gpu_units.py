"""Unit encoding (2048 elements per wave) at the sizes where it can go wrong:
edges of segments, units, superblocks and rounds, payloads held in LDS and
payloads too large to be held, workers past the end of many short jobs, and
the fp64 quotient by reciprocal and corrections.  Everything is compared bit
for bit with the CPU oracle or with IEEE division.
"""
import sys

import numpy as np
import pytest

from paper_2308_05199_amd import synth

pytestmark = pytest.mark.gpu

UNIT, ROUND, ROUND_FUSED = 2048, 15 * 2048, 11 * 2048


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gz():
    import torch
    from paper_2308_05199_amd import gzccl
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return gzccl


@pytest.fixture(scope="module")
def ctx(gz):
    c = gz.Context(0, max_elems=1 << 25, max_requests=4096)
    yield c
    c.close()


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def field(kind, n, dt, seed):
    """smooth: small payloads; dense: wide planes, hardly held or not at all;
    raw: every block fails; mixed: all of them in turn."""
    g = np.random.default_rng(seed)
    x = synth.sinusoids(max(n, 1), seed=seed)[:n].astype(dt)
    dense = g.uniform(-2000.0, 2000.0, n).astype(dt)
    if kind == "dense":
        return dense
    if kind == "raw":
        x[::17] = np.nan
        return x
    if kind == "mixed":
        for lo in range(0, n, 3000):
            x[lo:lo + 700] = dense[lo:lo + 700]
        x[5::9001] = np.inf
    return x


SIZES = [1, 2047, 2048, 2049, 4095, 4097, 3 * UNIT - 1, 3 * UNIT + 1, ROUND - 1, ROUND,
         ROUND + 33, 3 * ROUND + UNIT + 5, 200 * 3 * UNIT + 7]


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("kind", ["smooth", "dense", "raw", "mixed"])
def test_compress_at_unit_edges(ctx, oracle, dt, L, kind):
    import torch
    for n in SIZES:
        say("units", dt.__name__, L, kind, n)
        x = field(kind, n, dt, n)
        out, nb = ctx.compress(dev(x), 1e-4, block_len=L)
        torch.cuda.synchronize()
        want = oracle.compress(x, 1e-4, block_len=L)
        assert out[:int(nb.item())].cpu().numpy().tobytes() == want.tobytes(), n
    assert ctx.device_status() == 0


@pytest.mark.parametrize("L", [32, 128])
@pytest.mark.parametrize("kind", ["smooth", "dense", "mixed"])
def test_fused_at_unit_edges(ctx, oracle, L, kind):
    import torch
    for n in (1, 2049, 4097, ROUND_FUSED - 1, ROUND_FUSED + 1, 5 * ROUND_FUSED + UNIT + 3,
              200 * 3 * UNIT + 7):
        say("fused units", L, kind, n)
        x, y = field(kind, n, np.float32, n), field(kind, n, np.float32, n + 1)
        s = oracle.compress(x, 1e-4, block_len=L)
        out, nb = ctx.fused_reduce_step(dev(s), dev(y), 1e-4, block_len=L)
        torch.cuda.synchronize()
        want = oracle.fused_step(s, y, 1e-4, block_len=L)
        assert out[:int(nb.item())].cpu().numpy().tobytes() == want.tobytes(), n
    assert ctx.device_status() == 0


@pytest.mark.parametrize("op", ["compress", "fused"])
def test_long_jobs_among_many_short_ones(gz, ctx, oracle, op):
    """Most workers are past the end of the short jobs for many rounds in a
    row while they hold a long job's units."""
    import torch
    g = np.random.default_rng(5)
    f64 = op == "compress"
    ns = [int(g.integers(1, 200)) for _ in range(3900)]
    for k in range(0, 3900, 50):
        ns[k] = int(g.integers(10 * UNIT, 20 * UNIT))
    xs = [field("smooth", n, np.float64 if f64 and k % 3 == 0 else np.float32, k)
          for k, n in enumerate(ns)]
    ys = [synth.sinusoids(n, seed=k + 1) for k, n in enumerate(ns)]
    ins = xs if op == "compress" else [oracle.compress(x, 1e-4) for x in xs]
    items = []
    for n, a, y in zip(ns, ins, ys):
        code = gz.GZ_F64 if a.dtype == np.float64 else gz.GZ_F32
        cap = gz.bound(n, code)
        items.append({"in": dev(a), "out": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                      "out_bytes": torch.zeros(1, dtype=torch.int64, device="cuda"), "n": n,
                      "out_cap": cap, "eb": 1e-4, "dtype": code,
                      **({"local": dev(y), "in_bytes": a.size} if op == "fused" else {})})
    say("many short jobs", op, len(ns), sum(ns))
    plan = ctx.plan(gz.GZ_OP_COMPRESS if op == "compress" else gz.GZ_OP_FUSED,
                    ctx.requests(items))
    for _ in range(2):
        plan.launch()
    torch.cuda.synchronize()
    assert ctx.device_status() == 0
    for k, (it, a, y) in enumerate(zip(items, ins, ys)):
        want = oracle.compress(a, 1e-4) if op == "compress" else oracle.fused_step(a, y, 1e-4)
        got = it["out"][:int(it["out_bytes"].item())].cpu().numpy()
        assert got.tobytes() == want.tobytes(), (k, ns[k])
    plan.close()


@pytest.mark.parametrize("eb", [1e-4, 1.0 / 3.0, 7e-301, 3e-280, 2.0 ** -900, 2.0 ** 880, 1e290])
def test_fp64_quotients_are_correctly_rounded(ctx, eb):
    """Quotients near halves and over the whole range, steps on both sides of
    the reciprocal's limits, against IEEE division."""
    import torch
    g = np.random.default_rng(9)
    t = 2.0 * eb
    n = 1 << 18
    q = np.concatenate([g.integers(-(1 << 29), 1 << 29, n).astype(np.float64) + 0.5,
                        np.exp(g.uniform(-3, 21, n)), g.integers(-9, 9, n) + 0.5])
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        x = q * t
        x = np.concatenate([x, np.nextafter(x, np.inf), np.nextafter(x, -np.inf),
                            [0.0, -0.0, np.nan, np.inf, -np.inf, 5e-324, 1.7e308]])
        say("fp64 quotients", eb, x.size)
        got_q, got_f = ctx.quantize(dev(x), eb)
        torch.cuda.synchronize()
        r = x / t
        rr = np.rint(r)
        fail = ~((np.abs(r) <= 536870911.0) & (np.abs(x - rr * t) <= eb))
        want = np.where(fail, 0.0, rr).astype(np.int64)
    assert np.array_equal(got_f.cpu().numpy() != 0, fail)
    assert np.array_equal(got_q.cpu().numpy().astype(np.int64), want)


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("L", [32, 64, 128])
@pytest.mark.parametrize("kind", ["smooth", "dense", "raw", "mixed"])
def test_decompress_at_unit_edges(ctx, oracle, dt, L, kind):
    """fp32 streams of 128 to 4096 superblocks and all fp64 streams are decoded
    by units; fp64 RAW payloads exceed the unit's LDS region."""
    import torch
    lo = 127 * 4096 if dt == np.float32 else 0
    for n in [lo + k for k in (1, 2047, 2048, 2049, 4095, 4096, 4097, 3 * UNIT + 33)]:
        say("decode units", dt.__name__, L, kind, n)
        s = oracle.compress(field(kind, n, dt, n), 1e-4, block_len=L)
        out = torch.full((n + 8,), -7.0, dtype=torch.float32 if dt == np.float32 else torch.float64,
                         device="cuda")
        ctx.decompress(dev(s), n, block_len=L, out=out[:n])
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert got[:n].tobytes() == oracle.decompress(s).tobytes(), n
        assert (got[n:] == -7.0).all(), n
    assert ctx.device_status() == 0


@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_malformed_units_set_the_status(gz, ctx, oracle, dt):
    """A damaged header byte, table entry or stream header is found whichever
    unit of the superblock holds it, in single streams and in batches."""
    import torch
    n = 130 * 4096 + 5
    s = oracle.compress(field("smooth", n, dt, 3), 1e-4)
    ns = (n + 4095) // 4096
    hb = 64 + 4 * ns
    tdt = torch.float32 if dt == np.float32 else torch.float64
    for what, at in (("first unit's header byte", hb + 128 * 7 + 3),
                     ("second unit's header byte", hb + 128 * 7 + 100), ("table", 64 + 4 * 9),
                     ("magic", 0), ("size", 8)):
        say("malformed", dt.__name__, what)
        b = s.copy()
        b[at] ^= 0x15
        ctx.decompress(dev(b), n, dtype=tdt)
        assert ctx.device_status() == gz.GZ_ECORRUPT, what
        x64 = oracle.compress(field("smooth", 5000, np.float64, 4), 1e-4)
        good = torch.zeros(5000, dtype=torch.float64, device="cuda")
        ctx.batch(gz.GZ_OP_DECOMPRESS, ctx.requests([
            {"in": dev(b), "in_bytes": b.size, "out": torch.zeros(n, dtype=tdt, device="cuda"),
             "n": n, "dtype": gz.GZ_F32 if dt == np.float32 else gz.GZ_F64},
            {"in": dev(x64), "in_bytes": x64.size, "out": good, "n": 5000, "dtype": gz.GZ_F64}]))
        assert ctx.device_status() == gz.GZ_ECORRUPT, what
        assert good.cpu().numpy().tobytes() == oracle.decompress(x64).tobytes(), what
    ctx.decompress(dev(s), n, dtype=tdt)
    assert ctx.device_status() == 0


@pytest.mark.parametrize("nx,rows", [(8, 8), (8, 264), (72, 40), (1024, 72)])
def test_tile_decode_at_unit_edges(gz, ctx, oracle, nx, rows):
    import ctypes
    import torch
    for kind in ("smooth", "mixed"):
        x = field(kind, nx * rows, np.float32, nx + rows)
        s = oracle.compress(x, 1e-4, block_len=64, mode=1, nx=nx, select=1)
        y = torch.zeros(x.size, device="cuda")
        S = dev(s)
        p = gz.gz_params(64, 0, 0, 1, 1, nx)
        say("tiles", nx, rows, kind)
        assert gz.gz_decompress(ctx.h, gz._ptr(S), s.size, x.size, gz.GZ_F32, ctypes.byref(p),
                                gz._ptr(y), gz._stream()) == gz.GZ_OK
        torch.cuda.synchronize()
        assert ctx.device_status() == 0
        assert y.cpu().numpy().tobytes() == oracle.decompress(s).tobytes()


@pytest.mark.parametrize("select", [1, 2])
@pytest.mark.parametrize("nx,rows", [(8, 8), (64, 32), (72, 40), (8, 264), (1024, 72), (2048, 360)])
def test_tile_compress_at_unit_edges(gz, ctx, oracle, select, nx, rows):
    """Units of 32 tiles: one tile, a whole unit, ragged rows of tiles, and more
    than one round; payloads held and not."""
    import torch
    from paper_2308_05199_amd import selector
    for kind in ("smooth", "dense", "raw", "mixed"):
        say("tile units", nx, rows, select, kind)
        x = field(kind, nx * rows, np.float32, nx * rows + select)
        out = torch.zeros(gz.bound(x.size, gz.GZ_F32, 64), dtype=torch.uint8, device="cuda")
        nb = torch.zeros(1, dtype=torch.int64, device="cuda")
        selector.tile_compress(ctx, dev(x), nx, 1e-4, select, out, nb)
        torch.cuda.synchronize()
        want = oracle.compress(x, 1e-4, block_len=64, mode=1, nx=nx, select=select)
        assert out[:int(nb.item())].cpu().numpy().tobytes() == want.tobytes()
    assert ctx.device_status() == 0


@pytest.mark.parametrize("kind", ["smooth", "dense"])
def test_good_jobs_among_malformed_ones(gz, ctx, oracle, kind):
    """Long runs of malformed one-unit jobs, whose workers wait for no offset,
    between good jobs of one and of several rounds: a run is longer than the
    rounds a workgroup keeps, and the good jobs' streams are whole."""
    import torch
    ns = [1500] * 4000
    for k in range(0, 4000, 397):
        ns[k] = 1500 + 11 * UNIT * (k // 397 % 3)
    good = [k % 397 == 0 or k % 131 == 7 or k == 3999 for k in range(4000)]
    xs = {n: (field(kind, n, np.float32, n), field(kind, n, np.float32, n + 1)) for n in set(ns)}
    s = {n: oracle.compress(x, 1e-4) for n, (x, _) in xs.items()}
    want = {n: oracle.fused_step(s[n], xs[n][1], 1e-4).tobytes() for n in xs}
    bad = s[1500].copy()
    bad[0] ^= 0x15  # the magic word
    S, Y, B = {n: dev(a) for n, a in s.items()}, {n: dev(y) for n, (_, y) in xs.items()}, dev(bad)
    sizes = torch.zeros(len(ns), dtype=torch.int64, device="cuda")
    items = []
    for k, n in enumerate(ns):
        cap = gz.bound(n)
        items.append({"in": S[n] if good[k] else B, "in_bytes": S[n].numel() if good[k] else bad.size,
                      "local": Y[n], "out": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                      "out_bytes": sizes[k:k + 1], "n": n, "out_cap": cap, "eb": 1e-4,
                      "dtype": gz.GZ_F32})
    say("good among malformed", kind, sum(good), "of", len(ns))
    for _ in range(2):
        sizes.zero_()
        ctx.batch(gz.GZ_OP_FUSED, ctx.requests(items))
        assert ctx.device_status() == gz.GZ_ECORRUPT
        got = sizes.cpu().numpy()
        for k, n in enumerate(ns):
            if good[k]:
                assert items[k]["out"][:int(got[k])].cpu().numpy().tobytes() == want[n], k
            else:
                assert got[k] == 0, k


@pytest.mark.parametrize("L", [32, 64, 128])
def test_empty_fused_step_ignores_what_follows(gz, ctx, oracle, L):
    """An empty stream (n = 0) at the start of a larger buffer with other bytes
    behind it, stated whole as readable: single calls on every kernel, a batch
    and a plan with other jobs beside it."""
    import torch
    s = oracle.compress(np.zeros(0, np.float32), 1e-4, block_len=L)
    want = oracle.fused_step(s, np.zeros(0, np.float32), 2e-4, block_len=L).tobytes()
    buf = np.full(400, 0xA7, np.uint8)
    buf[:s.size] = s
    x, y = field("smooth", 5000, np.float32, 1), field("smooth", 5000, np.float32, 2)
    t = oracle.compress(x, 1e-4, block_len=L)
    want_t = oracle.fused_step(t, y, 2e-4, block_len=L).tobytes()
    B, T, Y, none = dev(buf), dev(t), dev(y), torch.zeros(0, device="cuda")
    for in_bytes in (64, 67, 68, 72, 400):
        for threads in (0, 64, 128, 256, 1024):
            say("empty fused", L, in_bytes, threads)
            out, nb = ctx.fused_reduce_step(B, none, 2e-4, block_len=L, in_bytes=in_bytes,
                                            threads=threads)
            assert ctx.device_status() == 0, (in_bytes, threads)
            assert out[:int(nb.item())].cpu().numpy().tobytes() == want, (in_bytes, threads)

    def items():
        r = []
        for n, a, ib, loc in ((0, B, 400, none), (5000, T, t.size, Y), (0, B, 400, none)):
            cap = gz.bound(n, gz.GZ_F32, L)
            r.append({"in": a, "in_bytes": ib, "local": loc, "n": n, "out_cap": cap, "eb": 2e-4,
                      "out": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                      "out_bytes": torch.zeros(1, dtype=torch.int64, device="cuda"),
                      "dtype": gz.GZ_F32, "block_len": L})
        return r

    for how in ("batch", "plan"):
        for sel, threads in ((slice(0, 3), 0), (slice(0, 1), 0), (slice(0, 3), 256)):
            it = items()[sel]
            say("empty fused", how, L, len(it), threads)
            if how == "batch":
                ctx.batch(gz.GZ_OP_FUSED, ctx.requests(it), threads=threads)
            else:
                plan = ctx.plan(gz.GZ_OP_FUSED, ctx.requests(it), threads=threads)
                plan.launch()
            assert ctx.device_status() == 0
            for k, q in enumerate(it):
                got = q["out"][:int(q["out_bytes"].item())].cpu().numpy().tobytes()
                assert got == (want_t if q["n"] else want), (how, k)
            if how == "plan":
                plan.close()


def patchy(n, dt, share, seed):
    """Runs of one unit, the given share of them dense (payloads too large to be
    held), the others smooth."""
    g = np.random.default_rng(seed)
    x = synth.sinusoids(n, seed=seed).astype(dt)
    for u in np.flatnonzero(g.random(n // UNIT) < share):
        x[u * UNIT:(u + 1) * UNIT] += g.uniform(-50.0, 50.0, UNIT).astype(dt)
    return x


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("share", [0.02, 0.5])
def test_large_payloads_between_small_ones(oracle, gz, dt, share):
    """Several rounds per workgroup, with payloads that are held and payloads
    that are not: single streams, and batches on both sides of the rule for
    early tickets."""
    import torch
    c = gz.Context(0, max_elems=3 << 24, max_requests=16)
    for n, L in ((1 << 24) + 777, 32), ((3 << 22) + UNIT, 64), ((1 << 23) + 4097, 128):
        say("patchy", dt.__name__, share, n, L)
        x = patchy(n, dt, share, n)
        want = oracle.compress(x, 1e-4, block_len=L, mt=True).tobytes()
        # fp32 streams of this size take strips by default, units when asked for
        for threads in (0, 64) if dt == np.float32 else (0,):
            out, nb = c.compress(dev(x), 1e-4, block_len=L, threads=threads)
            torch.cuda.synchronize()
            assert out[:int(nb.item())].cpu().numpy().tobytes() == want, (n, L, threads)
    for jobs, n in ((8, (1 << 20) + 5), (12, (1 << 22) + 3)):
        code = gz.GZ_F32 if dt == np.float32 else gz.GZ_F64
        xs = [patchy(n, dt, share, k) for k in range(3)]
        want = [oracle.compress(x, 1e-4, mt=True).tobytes() for x in xs]
        D, cap = [dev(x) for x in xs], gz.bound(n, code)
        sizes = torch.zeros(jobs, dtype=torch.int64, device="cuda")
        items = [{"in": D[k % 3], "out": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                  "out_bytes": sizes[k:k + 1], "n": n, "out_cap": cap, "eb": 1e-4, "dtype": code}
                 for k in range(jobs)]
        say("patchy batch", dt.__name__, share, jobs, n)
        for _ in range(2):
            c.batch(gz.GZ_OP_COMPRESS, c.requests(items))
        assert c.device_status() == 0
        for k, it in enumerate(items):
            assert it["out"][:int(sizes[k].item())].cpu().numpy().tobytes() == want[k % 3], (jobs, k)
    c.close()


@pytest.mark.parametrize("op", ["compress", "fused"])
@pytest.mark.parametrize("jobs,n", [(900, 1 * UNIT), (700, 3 * UNIT), (500, 3 * UNIT + 1),
                                    (400, 7 * UNIT), (300, 7 * UNIT + 1), (1100, 3 * UNIT)])
def test_batches_of_equal_short_jobs(gz, ctx, oracle, op, jobs, n):
    """Rounds of 3, 7 or all workers, one round per job or two, one round per
    workgroup or several; every third compression job is fp64, one size less."""
    import torch
    xs = [field("mixed", n - (k % 3 == 2), np.float64 if op == "compress" and k % 3 == 2
                else np.float32, k) for k in range(6)]
    ys = [field("smooth", x.size, np.float32, k + 9) for k, x in enumerate(xs)]
    if op == "fused":
        xs = [oracle.compress(x, 1e-4) for x in xs]
        want = [oracle.fused_step(x, y, 1e-4).tobytes() for x, y in zip(xs, ys)]
    else:
        want = [oracle.compress(x, 1e-4).tobytes() for x in xs]
    X, Y = [dev(x) for x in xs], [dev(y) for y in ys]
    sizes = torch.zeros(jobs, dtype=torch.int64, device="cuda")
    items = []
    for k in range(jobs):
        i, m = k % 6, ys[k % 6].size
        code = gz.GZ_F64 if xs[i].dtype == np.float64 else gz.GZ_F32
        cap = gz.bound(m, code)
        items.append({"in": X[i], "out": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
                      "out_bytes": sizes[k:k + 1], "n": m, "out_cap": cap, "eb": 1e-4,
                      "dtype": code, **({"local": Y[i], "in_bytes": xs[i].size}
                                        if op == "fused" else {})})
    say("short jobs", op, jobs, n)
    for _ in range(2):
        ctx.batch(gz.GZ_OP_COMPRESS if op == "compress" else gz.GZ_OP_FUSED, ctx.requests(items))
    assert ctx.device_status() == 0
    for k, it in enumerate(items):
        assert it["out"][:int(sizes[k].item())].cpu().numpy().tobytes() == want[k % 6], k


@pytest.mark.parametrize("L", [32, 64, 128])
def test_long_fused_streams(ctx, oracle, gz, L):
    """Streams on both sides of one pass of the unit workers (256 CUs x 11 units),
    at edges of superblocks and rounds of eight; a damaged one sets the status."""
    import torch
    edge = 256 * 11 * UNIT
    for n, kind in ((edge, "mixed"), (edge + 1, "smooth"), (edge + 4097, "mixed"),
                    (edge + 8 * 4096 - 1, "raw")):
        say("long fused", L, n, kind)
        x, y = field(kind, n, np.float32, 3), field("smooth", n, np.float32, 4)
        s = oracle.compress(x, 1e-4, block_len=L, mt=True)
        want = oracle.fused_step(s, y, 1e-4, block_len=L, mt=True).tobytes()
        S, Y = dev(s), dev(y)
        for threads in (0, 64):
            out, nb = ctx.fused_reduce_step(S, Y, 1e-4, block_len=L, threads=threads)
            assert ctx.device_status() == 0
            assert out[:int(nb.item())].cpu().numpy().tobytes() == want, (n, threads)
    b = s.copy()
    b[64 + 4 * 700] ^= 0x15  # a table word
    ctx.fused_reduce_step(dev(b), Y, 1e-4, block_len=L)
    assert ctx.device_status() == gz.GZ_ECORRUPT
    out, nb = ctx.fused_reduce_step(S, Y, 1e-4, block_len=L)
    assert ctx.device_status() == 0
    assert out[:int(nb.item())].cpu().numpy().tobytes() == want


@pytest.mark.parametrize("L", [32, 64, 128])
def test_fused_raw_input_at_unit_edges(ctx, oracle, L):
    """Incoming streams of RAW blocks only, sums that are coded and sums that stay RAW."""
    for n in (1, 33, 2047, 2049, 4097, 3 * UNIT + 31, ROUND_FUSED + 5):
        x = field("smooth", n, np.float32, n)
        x[::8] = np.float32(3e38)
        for y in (-x, field("raw", n, np.float32, n + 1), field("smooth", n, np.float32, n + 2)):
            say("raw fused", L, n)
            s = oracle.compress(x, 1e-4, block_len=L)
            out, nb = ctx.fused_reduce_step(dev(s), dev(y), 1e-4, block_len=L)
            want = oracle.fused_step(s, y, 1e-4, block_len=L)
            assert ctx.device_status() == 0
            assert out[:int(nb.item())].cpu().numpy().tobytes() == want.tobytes(), n


@pytest.mark.parametrize("jobs,n", [(256, 1 << 15), (300, 1 << 15), (64, 1 << 17), (8, 1 << 20),
                                    (300, (1 << 15) - UNIT), (40, (1 << 16) + 3)])
def test_batches_on_both_sides_of_the_strip_rule(gz, ctx, oracle, jobs, n):
    """fp32 batches that strips divide better than rounds of units, and their
    neighbours that units take, by batch and by plan."""
    import torch
    xs = [field(k, n, np.float32, 5) for k in ("smooth", "mixed", "dense")]
    want = [oracle.compress(x, 1e-4).tobytes() for x in xs]
    D, cap = [dev(x) for x in xs], gz.bound(n)
    sizes = torch.zeros(jobs, dtype=torch.int64, device="cuda")
    items = [{"in": D[k % 3], "out": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
              "out_bytes": sizes[k:k + 1], "n": n, "out_cap": cap, "eb": 1e-4,
              "dtype": gz.GZ_F32} for k in range(jobs)]
    reqs = ctx.requests(items)
    say("strip rule", jobs, n)
    plan = ctx.plan(gz.GZ_OP_COMPRESS, reqs)
    for run in (lambda: ctx.batch(gz.GZ_OP_COMPRESS, reqs), plan.launch):
        sizes.zero_()
        run()
        assert ctx.device_status() == 0
        for k, it in enumerate(items):
            assert it["out"][:int(sizes[k].item())].cpu().numpy().tobytes() == want[k % 3], k
    plan.close()


@pytest.mark.parametrize("eb", [5e-324, 1e-310, 2.0 ** -1023, 1e-290, 2.0 ** -902, 2.0 ** 900,
                                1e300, 8e307])
def test_fp64_steps_out_of_the_reciprocals_range(ctx, oracle, eb):
    """Strips scale such steps by a power of two, units divide: the oracle's bytes
    from both, for quotients near halves, over the whole range and failing ones."""
    import torch
    g = np.random.default_rng(21)
    n = 40000
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        x = np.concatenate([g.integers(-300, 300, n) + 0.5, g.integers(-40, 40, n) + 0.5,
                            np.exp(g.uniform(-3, 21, n)), g.uniform(-4, 4, n)]) * (2.0 * eb)
        x = np.concatenate([x, np.nextafter(x, np.inf), np.nextafter(x, -np.inf),
                            [0.0, -0.0, np.inf, np.nan, 1.7e308, -1.7e308, 5e-324, 1.0, 2.0 ** 424]])
    want = oracle.compress(x, eb).tobytes()
    for threads in (0, 128, 256):
        say("steps out of range", eb, threads)
        out, nb = ctx.compress(dev(x), eb, threads=threads)
        assert ctx.device_status() == 0
        assert out[:int(nb.item())].cpu().numpy().tobytes() == want, threads
