"""Batched engine and continuous batching (serving) against the oracle.

Each request is an H-equation solve (eq. (3.2), x0 = ones) by Algorithm 2.1
with an FP16 LU and IR.  Acceptance per request is the same as for a single
solve: the final iterate within 1e-9 (relative) of the oracle's solution and
the oracle's FP64 Newton iteration count or one more.  A request's result
must not depend on what else is in the batch: alone and in a mix the result
is bitwise identical.
"""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import serving_stream

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2307_16051_amd as n3p
    assert torch.cuda.is_available()
    return n3p, torch


_ORC = {}


def oracle_ref(n, c):
    """(Picard solution, FP64 Newton count) from the oracle, cached per (n, c)."""
    key = (n, round(c, 12))
    if key not in _ORC:
        its = O.newton_heq(n, c, floor=False).its
        _ORC[key] = (O.heq_picard(n, c, tol=1e-15), its)
    return _ORC[key]


def rel_err(x, ref):
    return float(np.linalg.norm(x - ref) / np.linalg.norm(ref))


def make_pool(n3p, torch, sizes, max_slots, prec=0):
    nbytes = n3p.engine_fixed_bytes(max_slots) + sum(n3p.engine_request_bytes(n, prec) for n in sizes)
    return torch.empty(nbytes + 4096, dtype=torch.uint8, device="cuda")


def run_to_completion(eng, slots, max_steps=40):
    for _ in range(max_steps):
        if all(eng.state(s)[0] == 3 for s in slots):
            return
        eng.step()
    raise AssertionError("requests did not finish in %d steps" % max_steps)


@pytest.mark.parametrize("prec", ["FP16", "BF16"])
def test_engine_batch_matches_oracle(env, prec):
    n3p, torch = env
    reqs = [(128, 0.5), (256, 0.9), (500, 0.99), (1000, 0.9), (1024, 0.99), (2048, 0.99)]
    print("case engine batch %s %s" % (prec, reqs), flush=True)
    p = getattr(n3p, prec)
    cfg = n3p.EngineConfig.default(max_slots=8, lu_prec=p)
    pool = make_pool(n3p, torch, [n for n, _ in reqs], 8, p)
    eng = n3p.Engine(pool, cfg)
    slots = [eng.admit(n, c) for n, c in reqs]
    assert None not in slots
    run_to_completion(eng, slots)
    for (n, c), s in zip(reqs, slots):
        x = torch.empty(n, dtype=torch.float64, device="cuda")
        rep = eng.collect(s, x)
        xr, its_ref = oracle_ref(n, c)
        err = rel_err(x.cpu().numpy(), xr)
        print("  n=%d c=%g its=%d (oracle %d) err=%.2e lin=%s" % (n, c, rep.its, its_ref, err,
                                                                  rep.lin_its), flush=True)
        assert rep.status == 0
        assert rep.its in (its_ref, its_ref + 1)
        assert err <= 1e-9
    eng.close()


def test_engine_matches_single_solve_path(env):
    """The batched engine and n3p_solve run the same method: same iteration
    count, the same solution to the rounding floor of the stopping rule."""
    n3p, torch = env
    n, c = 777, 0.99
    cfg = n3p.EngineConfig.default(max_slots=2)
    eng = n3p.Engine(make_pool(n3p, torch, [n], 2), cfg)
    s = eng.admit(n, c)
    run_to_completion(eng, [s])
    xb = torch.empty(n, dtype=torch.float64, device="cuda")
    rb = eng.collect(s, xb)
    xs, rs = n3p.solve_heq(n, c)
    assert rb.its == rs.its
    np.testing.assert_allclose(rb.resid_rel[1:4], rs.resid_rel[1:4], rtol=1e-3)
    assert rel_err(xb.cpu().numpy(), xs.cpu().numpy()) <= 1e-9
    eng.close()


def test_result_identical_alone_and_in_mix(env):
    """Continuous batching must not change a request's arithmetic."""
    n3p, torch = env
    target = (1000, 0.95)
    cfg = n3p.EngineConfig.default(max_slots=8)
    others = [(2048, 0.99), (512, 0.6), (128, 0.999), (1500, 0.9), (256, 0.8), (640, 0.97)]
    pool = make_pool(n3p, torch, [target[0]] + [n for n, _ in others], 8)

    eng = n3p.Engine(pool, cfg)
    s = eng.admit(*target)
    run_to_completion(eng, [s])
    x_alone = torch.empty(target[0], dtype=torch.float64, device="cuda")
    r_alone = eng.collect(s, x_alone)
    eng.close()

    eng = n3p.Engine(pool, cfg)
    live = [eng.admit(*others[0]), eng.admit(*others[1])]
    eng.step()                      # the target joins a batch already under way
    s = eng.admit(*target)
    eng.step()
    live += [eng.admit(*others[2]), eng.admit(*others[3])]
    eng.step()
    live += [eng.admit(*others[4]), eng.admit(*others[5])]
    assert None not in live
    run_to_completion(eng, live + [s])
    x_mix = torch.empty(target[0], dtype=torch.float64, device="cuda")
    r_mix = eng.collect(s, x_mix)
    for k in live:
        eng.collect(k, None)
    eng.close()
    print("  alone its=%d mix its=%d" % (r_alone.its, r_mix.its), flush=True)
    assert r_alone.status == r_mix.status == 0
    assert r_alone.its == r_mix.its
    assert r_alone.resid_rel == r_mix.resid_rel
    assert torch.equal(x_alone, x_mix)


def test_serve_stream_continuous_batching(env):
    """A seeded Poisson stream through n3p_serve: every result checked."""
    n3p, torch = env
    reqs = serving_stream(count=48, rate_per_s=400.0, seed=11, sizes=(128, 256, 512))
    ns = [r.n for r in reqs]
    cs = [r.c for r in reqs]
    ts = [r.arrival_s for r in reqs]
    off = np.concatenate([[0], np.cumsum(ns)[:-1]]).tolist()
    x_out = torch.zeros(int(sum(ns)), dtype=torch.float64, device="cuda")
    cfg = n3p.EngineConfig.default(max_slots=16, max_n=512)
    pool = make_pool(n3p, torch, [512] * 16, 16)
    its, status, lat, stats = n3p.serve(ns, cs, ts, pool, cfg, x_out=x_out, x_off=off)
    print("  stats %s" % stats, flush=True)
    assert all(s == 0 for s in status)
    assert stats["max_active"] > 1          # requests overlapped on the device
    assert 0 < stats["p50_ms"] <= stats["p99_ms"] <= stats["max_ms"]
    assert stats["solves_per_s"] > 0
    xs = x_out.cpu().numpy()
    for i, (n, c) in enumerate(zip(ns, cs)):
        xr, its_ref = oracle_ref(n, c)
        assert its[i] in (its_ref, its_ref + 1), (i, n, c, its[i], its_ref)
        assert rel_err(xs[off[i]:off[i] + n], xr) <= 1e-9, (i, n, c)


def test_admission_is_bounded_by_the_pool(env):
    """A pool that holds two requests: the rest wait, all finish."""
    n3p, torch = env
    n = 512
    cfg = n3p.EngineConfig.default(max_slots=8, max_n=n)
    pool = make_pool(n3p, torch, [n, n], 8)
    its, status, lat, stats = n3p.serve([n] * 6, [0.9] * 6, [0.0] * 6, pool, cfg)
    print("  stats %s" % stats, flush=True)
    assert all(s == 0 for s in status)
    assert stats["max_active"] == 2
    _, its_ref = oracle_ref(n, 0.9)
    assert all(k in (its_ref, its_ref + 1) for k in its)


def test_engine_rejects_when_full(env):
    n3p, torch = env
    cfg = n3p.EngineConfig.default(max_slots=2, max_n=256)
    eng = n3p.Engine(make_pool(n3p, torch, [256, 256, 256], 2), cfg)
    assert eng.admit(256, 0.9) is not None
    assert eng.admit(256, 0.9) is not None
    assert eng.admit(256, 0.9) is None         # no free slot
    with pytest.raises(n3p.N3PError):
        eng.admit(4096, 0.9)                   # above max_n
    eng.close()


def test_autotune_then_solve(env):
    n3p, torch = env
    reqs = [(1024, 0.9)] * 4 + [(512, 0.99)] * 4
    cfg = n3p.EngineConfig.default(max_slots=8, max_n=1024)
    eng = n3p.Engine(make_pool(n3p, torch, [n for n, _ in reqs], 8), cfg)
    slots = [eng.admit(n, c) for n, c in reqs]
    best, ms = eng.autotune()
    print("  autotune best %s, %d candidates, %.3f..%.3f ms" % (best.as_dict(), len(ms), min(ms),
                                                               max(ms)), flush=True)
    assert len(ms) == 24 and all(v > 0 for v in ms)
    run_to_completion(eng, slots)
    for (n, c), s in zip(reqs, slots):
        x = torch.empty(n, dtype=torch.float64, device="cuda")
        rep = eng.collect(s, x)
        xr, its_ref = oracle_ref(n, c)
        assert rep.status == 0 and rep.its in (its_ref, its_ref + 1)
        assert rel_err(x.cpu().numpy(), xr) <= 1e-9
    eng.close()


@pytest.mark.parametrize("count", [64, 65, 130])
def test_engine_more_slots_than_a_wavefront(env, count):
    """The items of a batched launch are counted 64 slots at a time: one full
    chunk, one slot over, and three chunks of slots of one to five leaves."""
    n3p, torch = env
    reqs = [([64, 65, 130, 257][i % 4], [0.5, 0.9, 0.99][i % 3]) for i in range(count)]
    print("case engine %d slots" % count, flush=True)
    cfg = n3p.EngineConfig.default(max_slots=count, max_n=512)
    eng = n3p.Engine(make_pool(n3p, torch, [n for n, _ in reqs], count), cfg)
    slots = [eng.admit(n, c) for n, c in reqs]
    assert None not in slots
    run_to_completion(eng, slots)
    for (n, c), s in zip(reqs, slots):
        x = torch.empty(n, dtype=torch.float64, device="cuda")
        rep = eng.collect(s, x)
        xr, its_ref = oracle_ref(n, c)
        assert rep.status == 0 and rep.its in (its_ref, its_ref + 1), (s, n, c)
        assert rel_err(x.cpu().numpy(), xr) <= 1e-9, (s, n, c)
    eng.close()


@pytest.mark.parametrize("prec", ["FP16", "BF16"])
def test_engine_small_requests_alone_and_beside_large_ones(env, prec):
    """Requests of up to 256 padded rows are solved by substitution, larger
    ones by blocks: sizes on both sides of the line and at the blocks' edges,
    first all small ones together (no launch for blocks), then beside requests
    of more rows, with the same bits."""
    n3p, torch = env
    p = getattr(n3p, prec)
    small = [(1, 0.9), (2, 0.5), (63, 0.9), (64, 0.99), (65, 0.9), (128, 0.99), (129, 0.5),
             (192, 0.9), (193, 0.99), (255, 0.9), (256, 0.99)]
    large = [(257, 0.9), (320, 0.99), (1000, 0.9)]
    print("case engine small requests %s" % prec, flush=True)
    xs = {}
    for reqs in (small, large, small + large):
        cfg = n3p.EngineConfig.default(max_slots=16, max_n=1024, lu_prec=p)
        eng = n3p.Engine(make_pool(n3p, torch, [n for n, _ in reqs], 16, p), cfg)
        slots = [eng.admit(n, c) for n, c in reqs]
        assert None not in slots
        run_to_completion(eng, slots)
        for (n, c), s in zip(reqs, slots):
            x = torch.empty(n, dtype=torch.float64, device="cuda")
            rep = eng.collect(s, x)
            xr, its_ref = oracle_ref(n, c)
            assert rep.status == 0 and rep.its in (its_ref, its_ref + 1), (n, c)
            assert rel_err(x.cpu().numpy(), xr) <= 1e-9, (n, c)
            if n in xs:
                assert torch.equal(x, xs[n]), (n, c)
            xs[n] = x
        eng.close()


@pytest.mark.parametrize("prec", ["FP16", "BF16"])
def test_engine_ill_conditioned_requests(env, prec):
    """c near one: the Jacobian nears singularity at the solution, refinement
    needs more sweeps, and the solves by blocks (explicit inverses of the
    diagonal blocks) have to carry it as substitution does."""
    n3p, torch = env
    reqs = [(200, 0.9999), (300, 0.9999), (512, 0.9999), (1024, 0.9999), (300, 0.99999), (1024, 0.99999)]
    print("case engine ill-conditioned %s" % prec, flush=True)
    p = getattr(n3p, prec)
    cfg = n3p.EngineConfig.default(max_slots=8, lu_prec=p)
    eng = n3p.Engine(make_pool(n3p, torch, [n for n, _ in reqs], 8, p), cfg)
    slots = [eng.admit(n, c) for n, c in reqs]
    run_to_completion(eng, slots)
    for (n, c), s in zip(reqs, slots):
        x = torch.empty(n, dtype=torch.float64, device="cuda")
        rep = eng.collect(s, x)
        ref = O.newton_heq(n, c)
        err = rel_err(x.cpu().numpy(), ref.x_floor)
        print("  n=%d c=%g its=%d (oracle %d) err=%.2e" % (n, c, rep.its, ref.its, err), flush=True)
        assert rep.status == 0 and rep.its in (ref.its, ref.its + 1), (n, c)
        assert err <= 1e-9, (n, c)
    eng.close()


@pytest.mark.parametrize("prec", ["FP16", "BF16"])
@pytest.mark.parametrize("n,c", [(320, 0.9), (512, 0.9999), (1024, 0.99999)])
def test_solve_by_blocks_is_as_accurate_as_substitution(env, prec, n, c):
    """One solve with half-precision factors of the Jacobian at the solution,
    by the row blocks that the engine and the single solves share, against 64
    bits with the same factors: no further off than row-by-row substitution
    in FP32."""
    n3p, torch = env
    J = torch.from_numpy(O.heq_jacobian(O.newton_heq(n, c).x_floor, c)).cuda()
    J = J * 2.0 ** torch.floor(9 - torch.log2(J.abs().amax(0)))[None, :]
    LU = J.t().contiguous().to({"FP16": torch.float16, "BF16": torch.bfloat16}[prec]).t()
    ipiv, info = n3p.getrf(LU)
    assert info == 0
    perm = torch.from_numpy(O.perm_from_ipiv(ipiv.cpu().numpy())).cuda()
    L64, A = LU.double(), LU.float()
    errs = {"blocks": [], "substitution": []}
    for seed in range(4):
        g = torch.Generator(device="cuda").manual_seed(seed)
        b = torch.randn(n, generator=g, device="cuda", dtype=torch.float32)
        ref = torch.linalg.solve_triangular(L64, b.double()[perm][:, None], upper=False, unitriangular=True)
        ref = torch.linalg.solve_triangular(L64, ref, upper=True)[:, 0]
        y = b[perm]
        for k in range(n - 1):
            y[k + 1:] = torch.addcmul(y[k + 1:], A[k + 1:, k], y[k], value=-1)
        for k in range(n - 1, -1, -1):
            y[k] = y[k] * (1.0 / A[k, k])
            y[:k] = torch.addcmul(y[:k], A[:k, k], y[k], value=-1)
        for name, x in (("blocks", n3p.getrs(LU, ipiv, b.clone())), ("substitution", y)):
            errs[name].append(float((x.double() - ref).norm() / ref.norm()))
    print("  %s n=%d c=%g error: blocks %.2e substitution %.2e" % (
        prec, n, c, np.mean(errs["blocks"]), np.mean(errs["substitution"])), flush=True)
    assert np.mean(errs["blocks"]) <= np.mean(errs["substitution"])
