"""Failure handling of the kernels' bounded waits, forced from the host.

With a wait bound of zero (gz_ctx_set_wait) every wait between waves that is
not satisfied at once expires: each encoding kernel (strips and per-wave,
single streams and batches, compression and the fused step) must still
finish and report either success with the oracle's bytes or GZ_ETIMEOUT.
With the default bound restored, the same calls are clean and bit-exact.
Every case prints its name before touching the GPU.
"""
import sys

import numpy as np
import pytest

from paper_2308_05199_amd import synth

pytestmark = pytest.mark.gpu


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
    c = gz.Context(0, max_elems=1 << 25, max_requests=64)
    yield c
    c.set_wait(1_000_000)
    c.close()


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


EB = 1e-4
N = (1 << 22) + 1234   # 1025 superblocks: 129 rounds, 129 strips of 32768


def _calls(gz, ctx, oracle):
    """(name, run() -> list of streams as numpy arrays, expected streams)."""
    import torch
    x = synth.sinusoids(N, seed=50)
    loc = np.random.default_rng(51).normal(0, 0.2, N).astype(np.float32)
    s = oracle.compress(x, EB)
    want_c = [s]
    want_f = [oracle.fused_step(s, loc, EB)]
    X, LOC, S = dev(x), dev(loc), dev(s)

    def compress(tpb):
        def run():
            out, nb = ctx.compress(X, EB, threads=tpb)
            torch.cuda.synchronize()
            return [out[:int(nb.item())].cpu().numpy()]
        return run

    def fused(tpb):
        def run():
            out, nb = ctx.fused_reduce_step(S, LOC, EB, threads=tpb)
            torch.cuda.synchronize()
            return [out[:int(nb.item())].cpu().numpy()]
        return run

    # a uniform batch of 4 fused requests (the per-wave batch kernel by default)
    cap = gz.bound(N)
    outs = [torch.empty(cap, dtype=torch.uint8, device="cuda") for _ in range(4)]
    nbs = [torch.zeros(1, dtype=torch.int64, device="cuda") for _ in range(4)]
    items = [{"in": S, "local": LOC, "out": o, "out_bytes": b, "n": N, "in_bytes": s.size,
              "out_cap": cap, "eb": EB, "dtype": gz.GZ_F32} for o, b in zip(outs, nbs)]
    reqs = ctx.requests(items)

    def batch(tpb):
        def run():
            ctx.batch(gz.GZ_OP_FUSED, reqs, threads=tpb)
            torch.cuda.synchronize()
            return [o[:int(b.item())].cpu().numpy() for o, b in zip(outs, nbs)]
        return run

    return [("compress strips", compress(1024), want_c),
            ("compress per-wave", compress(64), want_c),
            ("fused strips", fused(1024), want_f),
            ("fused per-wave", fused(64), want_f),
            ("fused batch per-wave", batch(64), want_f * 4),
            ("fused batch strips", batch(1024), want_f * 4)]


def test_zero_wait_bound_finishes_and_reports(gz, ctx, oracle):
    statuses = []
    for name, run, want in _calls(gz, ctx, oracle):
        say("zero wait bound:", name)
        ctx.set_wait(0)
        got = run()
        st = ctx.device_status()
        statuses.append(st)
        assert st in (gz.GZ_OK, gz.GZ_ETIMEOUT), (name, st)
        if st == gz.GZ_OK:
            assert all(g.tobytes() == w.tobytes() for g, w in zip(got, want)), name
        say("  status", st)
        ctx.set_wait(1_000_000)
        ctx.reset()
        say("default bound:", name)
        got = run()
        assert ctx.device_status() == gz.GZ_OK, name
        assert all(g.tobytes() == w.tobytes() for g, w in zip(got, want)), name
    say("statuses under the zero bound", statuses)


def _unit_calls(gz, c, oracle):
    """Unit launches of several rounds per workgroup, and the long fused step:
    (name, run, wanted)."""
    import torch
    from paper_2308_05199_amd import selector
    n = (1 << 20) + 77
    xs = [synth.sinusoids(n + 5000 * k, seed=k).astype(np.float64 if k % 2 else np.float32)
          for k in range(12)]
    xs[3][::64] = np.nan  # payloads too large to be held
    ss = [oracle.compress(x.astype(np.float32), EB) for x in xs[:6]]
    ys = [synth.sinusoids(x.size, seed=40 + k) for k, x in enumerate(xs[:6])]

    def batch(op, ins, ns, dts, extra):
        outs, nbs, items = [], [], []
        for k, (a, m, dt) in enumerate(zip(ins, ns, dts)):
            cap = gz.bound(m, dt)
            outs.append(torch.zeros(cap, dtype=torch.uint8, device="cuda"))
            nbs.append(torch.zeros(1, dtype=torch.int64, device="cuda"))
            items.append({"in": dev(a), "out": outs[-1], "out_bytes": nbs[-1], "n": m,
                          "out_cap": cap, "eb": EB, "dtype": dt, **extra(k)})
        reqs = c.requests(items)

        def run(keep=items):
            c.batch(op, reqs)
            torch.cuda.synchronize()
            return [o[:int(b.item())].cpu().numpy() for o, b in zip(outs, nbs)]
        return run

    calls = [("mixed compression batch",
              batch(gz.GZ_OP_COMPRESS, xs, [x.size for x in xs],
                    [gz.GZ_F64 if k % 2 else gz.GZ_F32 for k in range(12)], lambda k: {}),
              [oracle.compress(x, EB, mt=True) for x in xs]),
             ("uneven fused batch",
              batch(gz.GZ_OP_FUSED, ss, [x.size for x in xs[:6]], [gz.GZ_F32] * 6,
                    lambda k: {"in_bytes": ss[k].size, "local": dev(ys[k])}),
              [oracle.fused_step(s, y, EB, mt=True) for s, y in zip(ss, ys)])]

    root = np.concatenate([x.astype(np.float64) for x in xs])
    counts = [root.size // 3, root.size // 2 - 11, root.size - root.size // 3 - root.size // 2 + 11]
    displs = [0, counts[0], counts[0] + counts[1]]
    R = dev(root)

    def scatter():
        out, nb, off = c.scatter_compress(R, counts, displs, EB)
        torch.cuda.synchronize()
        o = out.cpu().numpy()
        b, f = nb.cpu().numpy().astype(int), off.cpu().numpy().astype(int)
        ok = all(0 <= f[k] <= o.size and 0 <= b[k] <= o.size - f[k] for k in range(3))
        return [o[f[k]:f[k] + b[k]] for k in range(3)] if ok else [o[:0]] * 3
    calls.append(("packed fp64 scatter", scatter,
                  [oracle.compress(root[d:d + m], EB, mt=True) for d, m in zip(displs, counts)]))

    tile = synth.sinusoids(2048 * 4096, seed=3)
    T = dev(tile)
    to = torch.zeros(gz.bound(tile.size, gz.GZ_F32, 64), dtype=torch.uint8, device="cuda")
    tn = torch.zeros(1, dtype=torch.int64, device="cuda")

    def tiles():
        selector.tile_compress(c, T, 2048, EB, 1, to, tn)
        torch.cuda.synchronize()
        return [to[:int(tn.item())].cpu().numpy()]
    calls.append(("tiles", tiles, [oracle.compress(tile, EB, block_len=64, mode=1, nx=2048,
                                                   select=1, mt=True)]))

    big = synth.sinusoids(1 << 23, seed=7)
    S, B = dev(oracle.compress(big, EB, mt=True)), dev(big)

    def long_fused():
        out, nb = c.fused_reduce_step(S, B, EB)
        torch.cuda.synchronize()
        return [out[:int(nb.item())].cpu().numpy()]
    calls.append(("long fused step", long_fused,
                  [oracle.fused_step(oracle.compress(big, EB, mt=True), big, EB, mt=True)]))
    return calls


def test_zero_wait_bound_on_unit_launches(gz, oracle):
    """A wait that expires ends the launch, and the next one, after a reset, is
    whole: batches of both kinds, a packed chain, tiles and the long fused step."""
    c = gz.Context(0, max_elems=1 << 25, max_requests=16)
    statuses = []
    for name, run, want in _unit_calls(gz, c, oracle):
        say("zero wait bound:", name)
        c.set_wait(0)
        got = run()
        st = c.device_status()
        statuses.append(st)
        assert st in (gz.GZ_OK, gz.GZ_ETIMEOUT), (name, st)
        if st == gz.GZ_OK:
            assert all(g.tobytes() == w.tobytes() for g, w in zip(got, want)), name
        c.set_wait(1_000_000)
        c.reset()
        say("default bound:", name, "after status", st)
        for _ in range(2):
            got = run()
            assert c.device_status() == gz.GZ_OK, name
            assert all(g.tobytes() == w.tobytes() for g, w in zip(got, want)), name
    say("statuses under the zero bound", statuses)
    c.close()
