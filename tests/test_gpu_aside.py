"""Work on the context's second stream (the refits beside a factorisation, E beside the one of M, the targets of the initialisation
beside that of H, a refit's right-hand side beside its own) and E in the launches of a small M's chain, against the same calls on a workspace that just does not hold both at a
time, and under capture: the same bits."""
import ctypes as C

import pytest
import torch

from paper_2510_03246_amd import inputs, strp

pytestmark = pytest.mark.gpu

NAMES = ("A", "Z", "W1", "W2", "score", "mask")


def _module(ctx, d, f, T, k, dtype="bf16", seed=5):
    cfg = inputs.WorkloadConfig("case", 1, d, f, 0, T, dtype, "t3", 3, 0.5, 1)
    m = inputs.make_ffn_module(cfg, 0, seed, "cuda", ld=(T + 7) // 8 * 8)
    return strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], T, k_max=k)


def _smallest(works):
    """smallest number of 256-byte granules for which works() holds"""
    lo, hi = 15, works.top
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if works(mid) else (mid, hi)
    return hi


class _Space:
    def __init__(self, ctx, nbytes, call, beside):
        self.ctx, self.call, self.beside = ctx, call, beside
        self.space = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.top = nbytes // 256

    def run(self, granules):
        """the call's result on that much workspace (None: refused), and whether it used the second stream"""
        ctx = self.ctx
        ctx.check(ctx.lib.strp_set_workspace(ctx.h, self.space.data_ptr(), granules * 256))
        ctx.profile_enable(True)
        got = self.call()
        names = [r[0] for r in ctx.profile_launches()]
        ctx.profile_enable(False)
        assert ctx.poll() == strp.OK
        return got, got is not None and self.beside(names)

    def __call__(self, granules):
        return self.run(granules)[1]


def _step_both_ways(d, f, T, k, mode, dtype, beside_by):
    """Two iterations each, at the full workspace, the least on which beside_by(the launches' names) holds, and 256 bytes below."""
    ctx = strp.Context(0)
    mod = _module(ctx, d, f, T, k, dtype)
    mod.init(strp.Params(1.0, 0.7, 0.01, mode, 1, k, 0))
    mod.Z += 0.25 * torch.randn(mod.Z.shape, generator=torch.Generator(device="cuda").manual_seed(k), device="cuda")
    mod.A.copy_(torch.relu(mod.Z))
    start = [t.clone() for t in (mod.Z, mod.A)]

    def call():
        for t, s in zip((mod.Z, mod.A), start):
            t.copy_(s)
        mod.state.sums_cached = mod.state.s = 0
        terms = []
        for _ in range(2):
            par, rep = strp.Params(1.0, 0.7, 0.01, mode, 1, k, 0), strp.Report()
            st = ctx.lib.strp_admm_step(ctx.h, C.byref(mod.desc), C.byref(mod.state), C.byref(par), C.byref(rep))
            if st != strp.OK:
                assert st == strp.ENOMEM
                return None
            terms.append(tuple(rep.terms))
        return [t.clone() for t in (mod.A[:, :T], mod.Z[:, :T], mod.W1, mod.W2, mod.score, mod.mask)] + [torch.tensor(terms)]      # what lies behind a row's tokens may be NaN

    w = _Space(ctx, ctx.workspace_bytes(mod.desc), call, beside_by)
    full, beside = w.run(w.top)
    assert beside
    least = _smallest(w)
    for granules, want in ((least, True), (least - 1, False)):
        got, beside = w.run(granules)
        assert beside == want and all(torch.equal(a, b) for a, b in zip(got, full)), (granules, want)
    ctx.close()


@pytest.mark.parametrize("d,f,T,k,mode,dtype", [(440, 1440, 9003, 600, strp.WANDA, "bf16"), (264, 1000, 30011, 401, strp.GAIN, "f32"), (72, 264, 70001, 131, strp.GAIN, "bf16"),
                                                (40, 160, 100000, 60, strp.WANDA, "f32"), (768, 1536, 2000, 1408, strp.WANDA, "bf16"), (256, 3072, 1024, 2000, strp.WANDA, "bf16")])
def test_step_beside_and_in_turn(d, f, T, k, mode, dtype):
    """Two iterations each.  The passes ride with the fc2 factorisation where the refits go in turn, and are a launch of their own beside it."""
    _step_both_ways(d, f, T, k, mode, dtype, lambda names: "pruned_rows" in names)


@pytest.mark.parametrize("d,f,T,k,mode,dtype", [(64, 256, 512, 128, strp.WANDA, "f32"), (40, 160, 333, 33, strp.GAIN, "f32"), (8, 64, 30011, 9, strp.WANDA, "bf16"),
                                                (200, 704, 1111, 301, strp.GAIN, "bf16"), (512, 1504, 513, 500, strp.WANDA, "f32")])
def test_residual_in_the_launches_of_the_chain(d, f, T, k, mode, dtype):
    """E, its turned plane, E E^T and the sum with M^-2 share the launches of M's chain where all are small, and go by themselves where there is no room."""
    _step_both_ways(d, f, T, k, mode, dtype, lambda names: not any(n.endswith("resid") for n in names))


@pytest.mark.parametrize("side,m,n,T", [(strp.SIDE_FC2, 333, 200, 20003), (strp.SIDE_FC2, 64, 1000, 10000), (strp.SIDE_FC2, 64, 1500, 20000), (strp.SIDE_FC2, 40, 2500, 5000), (strp.SIDE_FC1, 300, 136, 30000)])
def test_refit_beside_and_in_turn(side, m, n, T):
    ctx = strp.Context(0)
    g = torch.Generator(device="cuda").manual_seed(n)
    ld = (T + 7) // 8 * 8
    fc2 = side == strp.SIDE_FC2
    lhs = torch.randn((m, ld), generator=g, device="cuda")
    rhs = torch.randn((n + 5, ld), generator=g, device="cuda").bfloat16()
    idx = torch.randperm(n + 5, generator=g, device="cuda")[:n].sort().values.int() if fc2 else torch.arange(m, dtype=torch.int32, device="cuda")
    rows = rhs[idx.long()] if fc2 else rhs[:n]
    x = rows[:, :T].float()
    G = (x @ x.T).contiguous()
    W = torch.zeros((m, n + 5) if fc2 else (m, n), device="cuda")
    chol = torch.empty((n, n), dtype=torch.float64, device="cuda")
    rmat = rhs if fc2 else rhs[:n]

    def call():
        st = ctx.lib.strp_refit(ctx.h, side, G.data_ptr(), n, 0.5, chol.data_ptr(), 0, lhs.data_ptr(), strp.F32, ld, rmat.data_ptr(), strp.BF16, ld, T, idx.data_ptr(),
                                n if fc2 else m, W.data_ptr(), m, W.shape[1])
        return [W.clone(), chol.clone()] if st == strp.OK else None

    w = _Space(ctx, 1 << 30, call, lambda names: names[0] == "chol_factor_f64")
    full, beside = w.run(w.top)
    assert beside
    least = _smallest(w)
    got, beside = w.run(least)
    assert beside and all(torch.equal(a, b) for a, b in zip(got, full))
    got, beside = w.run(least - 1)
    assert not beside and all(torch.equal(a, b) for a, b in zip(got, full))
    ref = torch.linalg.solve(G.double() + 0.5 * torch.eye(n, dtype=torch.float64, device="cuda"), (lhs[:, :T].double() @ rmat[idx.long() if fc2 else slice(None)][:, :T].double().T).T).T
    kept = full[0][:, idx.long()] if fc2 else full[0]
    assert float((kept - ref).norm() / ref.norm()) <= 1e-4
    ctx.close()


@pytest.mark.parametrize("d,f,T,shift", [(136, 520, 3001, 0), (200, 704, 1003, 8), (520, 1040, 4000, 0)])
def test_initialisation_beside_and_in_turn(d, f, T, shift):
    """shift: bytes by which the factor's place is off a 16-byte boundary (it is then made in scratch and copied)"""
    ctx = strp.Context(0)
    mod = _module(ctx, d, f, T, f, "f32")
    room = torch.empty(8 * d * d + 16, dtype=torch.uint8, device="cuda")
    mod.state.cholH = room.data_ptr() + shift
    par = strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, f, 0)

    def call():
        st = ctx.lib.strp_module_init(ctx.h, C.byref(mod.desc), C.byref(mod.state), C.byref(par))
        return [t.clone() for t in (mod.Z, mod.A, mod.Y, mod.H, room[shift:shift + 8 * d * d], mod.scalars)] if st == strp.OK else None

    w = _Space(ctx, ctx.workspace_bytes(mod.desc), call, lambda names: "chol_factor_f64" in names and names.index("chol_factor_f64") < len(names) - 2 and
               any(n.endswith("initz") for n in names[names.index("chol_factor_f64"):]))
    full, beside = w.run(w.top)
    assert beside
    least = _smallest(w)
    got, beside = w.run(least)
    assert beside and all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, full))
    got, beside = w.run(least - 1)
    assert not beside and all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, full))
    ctx.close()


def test_captured_step_replays_as_the_eager_one():
    """A captured iteration holds both streams.  Every replay is one more iteration: the same bits as the eager ones, with other work and
    waits between them."""
    d, f, T, k = 264, 800, 9003, 300
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx, twin = strp.Context(0), strp.Context(0)
        mods = [_module(c, d, f, T, k) for c in (ctx, twin)]
        p = strp.Params(1.0, 0.7, 0.01, strp.GAIN, 1, k, 0)
        for mod in mods:
            mod.init(p)
            mod.state.sums_cached = 0
            mod.step(p, False)
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    mod, eager = mods
    with torch.cuda.graph(graph, stream=s):
        mod.step(p, False)
    for _ in range(4):
        with torch.cuda.stream(s):
            graph.replay()
            eager.step(p, False)
        torch.cuda.synchronize()
        assert all(torch.equal(getattr(mod, n), getattr(eager, n)) for n in NAMES)
    assert ctx.poll() == strp.OK and twin.poll() == strp.OK
    ctx.close()
    twin.close()


def test_contexts_on_streams_of_their_own():
    """Iterations of two modules interleaved on two streams, each with its second one: the same bits as alone."""
    shapes = [(264, 800, 9003, 300), (440, 1000, 5003, 420)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    p = [strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, sh[3], 0) for sh in shapes]

    def make(i):
        with torch.cuda.stream(streams[i]):
            mod = _module(strp.Context(0), *shapes[i])
            mod.init(p[i])
        return mod

    both, alone = [make(0), make(1)], [make(0), make(1)]
    torch.cuda.synchronize()
    for _ in range(3):
        for i in (0, 1):
            with torch.cuda.stream(streams[i]):
                both[i].step(p[i], False)
    torch.cuda.synchronize()
    for i in (0, 1):
        for _ in range(3):
            with torch.cuda.stream(streams[i]):
                alone[i].step(p[i], False)
            torch.cuda.synchronize()
    for a, b in zip(both, alone):
        assert all(torch.equal(getattr(a, n), getattr(b, n)) for n in NAMES)
        assert a.ctx.poll() == strp.OK


@pytest.mark.parametrize("m,n,T", [(64, 1000, 10000), (333, 4100, 4001), (16, 5320, 3000)])
def test_first_call_captured(m, n, T):
    """A context makes its second stream with the first call that can use it, but not while that is captured, which then goes in turn: the same bits as of
    the eager call that has it, also where the system takes launches per panel (63 to 68 and 84 to 90 tiles)."""
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx, twin = strp.Context(0, 1 << 30), strp.Context(0, 1 << 30)
        g = torch.Generator(device="cuda").manual_seed(n)
        ld = (T + 7) // 8 * 8
        lhs, rhs = (torch.randn((rows, ld), generator=g, device="cuda") for rows in (m, n))
        G = rhs[:, :T] @ rhs[:, :T].T
        idx = torch.arange(n, dtype=torch.int32, device="cuda")
        out = [[torch.zeros((m, n), device="cuda"), torch.zeros((n, n), dtype=torch.float64, device="cuda")] for _ in (0, 1)]
        call = lambda c, o: c.strp_refit(strp.SIDE_FC2, G, 0.01 * T, lhs, rhs, T, idx, o[0], chol=o[1])
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        call(ctx, out[0])
    with torch.cuda.stream(s):
        for _ in range(3):
            for t in out[0]:
                t.zero_()
            graph.replay()
            call(twin, out[1])
            torch.cuda.synchronize()
            assert ctx.poll() == strp.OK and twin.poll() == strp.OK
            assert all(torch.equal(a, b) for a, b in zip(*out))
    ctx.close()
    twin.close()
