"""GPU parity of the device walker (ndvm_walk_*) against the oracle, through
the C ABI: the structural walk on the device, no tape, no scheduling.

Random expression programs (ragged lane counts, many programs per launch),
the scalar benchmark programs, branch populations whose waves decide alike
or split (every arm walked under its lane mask, arms no lane takes
skipped), nested branches and loops, the edge cases of the adjoint table
(clamps, |x| at 0, NaN predicates), error paths, and the whole random-program
population at its benchmark size on sampled lanes."""
import numpy as np
import pytest

from conftest import record
from parity import judge
from wide_cases import chain, held_values
from workloads import bytecode as B
from workloads import configs
from workloads.bytecode import Asm

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_03574_amd as m
    return m


def walk(nd, programs, params, obs):
    """params: [n_prog, L, Pmax] numpy; returns loss [n_prog, L], grad."""
    ws = nd.walk_prepare(programs)
    p = torch.tensor(np.ascontiguousarray(params), device="cuda")
    o = torch.tensor(np.asarray(obs, dtype=np.float64), device="cuda")
    need = nd.walk_workspace_bytes(ws, p.shape[1])
    work = torch.empty(max(need, 8), dtype=torch.uint8, device="cuda")
    loss, grad = nd.walk_grad(ws, p, o, workspace=work)
    nd.walk_status(work)
    torch.cuda.synchronize()
    return loss.cpu().numpy(), grad.cpu().numpy()


def judge_all(oracle_mod, programs, n_params, params, obs, loss, grad, name):
    tot = dict(n_lanes=0, n_strict=0, n_ill_conditioned=0, n_libm_sensitive=0, n_other_arm=0)
    for q, bc in enumerate(programs):
        P = n_params[q]
        r = judge(oracle_mod, bc, params[q][:, :P], obs, loss[q], grad[q][:, :P])
        for k in tot:
            tot[k] += r[k]
    record(name, **tot)
    return tot


@pytest.mark.parametrize("L,seed", [(200, 1), (64, 2), (1, 3), (130, 4)])
def test_random_programs(nd, oracle_mod, L, seed):
    w = configs.random_programs(n_prog=48, L=L, n=16, seed=seed)
    loss, grad = walk(nd, w.programs, w.params, w.obs)
    tot = judge_all(oracle_mod, w.programs, w.n_params_each, w.params, w.obs, loss, grad, "walk_random")
    assert tot["n_lanes"] == 48 * L


def test_program_at_the_lds_limit(nd, oracle_mod):
    """The most structural state the validator accepts: its launch asks for the
    most LDS, some 70 KiB a wave."""
    from test_walk_host import at_the_lds_limit
    bc = at_the_lds_limit()
    p = np.random.default_rng(5).normal(size=(65, 63))
    loss, grad = walk(nd, [bc], p[None], np.zeros(0))
    r = judge(oracle_mod, bc, p, np.zeros(0), loss[0], grad[0])
    assert r["n_strict"] == 65


@pytest.mark.parametrize("name,kw", [("exp_decay", {}), ("logistic_euler", dict(L=300)),
                                     ("lotka_volterra_rk4", dict(L=130, T=40))])
def test_benchmark_programs(nd, oracle_mod, name, kw):
    w = configs.build(name, **kw)
    loss, grad = walk(nd, [w.bytecode], w.params[None], w.obs)
    r = judge(oracle_mod, w.bytecode, w.params, w.obs, loss[0], grad[0])
    record("walk_benchmark_program", workload=name, **r)
    # the same values the scheduled replay gives, within the bar
    tape = nd.tape_upload(nd.tape_build(w.bytecode))
    lt, gt = nd.grad(tape, torch.tensor(w.params, device="cuda"), torch.tensor(w.obs, device="cuda"))
    from parity import compare
    compare(loss[0], grad[0], lt.cpu().numpy(), gt.cpu().numpy())


@pytest.mark.parametrize("case", range(len(configs.BRANCH_TREES)))
@pytest.mark.parametrize("order", ["sorted", "mixed", "all_then", "all_else"])
def test_branch_populations(nd, oracle_mod, case, order):
    w = configs.branch_population(case, L=1000, n=16, order=order)
    loss, grad = walk(nd, [w.bytecode], w.params[None], w.obs)
    r = judge(oracle_mod, w.bytecode, w.params, w.obs, loss[0], grad[0])
    record("walk_branch_population", case=case, order=order, **r)


def test_nested_branches_loops_and_locals(nd, oracle_mod):
    # a loop whose body branches on the loop's observation, arms that write
    # locals, a nested branch on a parameter, stack shuffles across the arms
    A = Asm(3, 16)
    A.push(0.0).storel(0).param(2).storel(1)
    A.loop(16)
    A.obs(0, 1).param(0).iflt()
    A.loadl(0).obs(0, 1).param(1).mul().sin().add().storel(0)
    A.param(1).param(2).iflt().loadl(1).push(0.5).mul().push(1.0).add().storel(1)
    A.else_().loadl(1).sin().push(2.0).add().storel(1).endif()
    A.else_()
    A.loadl(0).obs(0, 1).param(0).sub().dup().mul().sub().storel(0)
    A.loadl(1).push(0.5).pow().storel(1)
    A.endif()
    A.endloop()
    A.loadl(0).loadl(1).swap().over().mul().add().halt()
    bc = A.bytes()
    rng = np.random.default_rng(3)
    obs = rng.uniform(-2, 2, 16)
    params = rng.uniform(0.1, 2, (777, 3))
    params[:, 0] = rng.uniform(-2.5, 2.5, 777)
    loss, grad = walk(nd, [bc], params[None], obs)
    r = judge(oracle_mod, bc, params, obs, loss[0], grad[0])
    record("walk_nested", **r)


def test_edge_programs(nd, oracle_mod):
    progs = [
        (Asm(3, 0).param(0).param(1).iflt().push(1000.0).param(2).mul().exp().else_().push(2.0)
         .param(2).mul().endif().halt().bytes(),
         [[1.0, 1.0, 5.0], [np.nan, 1.0, 5.0], [0.5, 1.0, 0.001], [2.0, 1.0, 5.0]]),
        (Asm(1, 0).param(0).log().halt().bytes(), [[1e-9], [-1.0], [1e-8], [2e-8]]),
        (Asm(1, 0).param(0).sqrt().halt().bytes(), [[1e-9], [4.0]]),
        (Asm(1, 0).param(0).abs().halt().bytes(), [[0.0], [-2.0], [3.0]]),
        (Asm(2, 0).param(1).halt().bytes(), [[3.0, 4.0]]),
        (Asm(2, 0).push(2.5).halt().bytes(), [[3.0, 4.0]]),
        (Asm(2, 0).param(0).param(1).pow().param(0).param(1).div().neg().add().cos().halt().bytes(),
         [[2.0, 0.5], [0.3, -1.5], [0.0, 2.0]]),
    ]
    for bc, params in progs:
        params = np.asarray(params, dtype=np.float64)
        lo, go, _ = oracle_mod.run(bc, params, [])
        loss, grad = walk(nd, [bc], params[None], [])
        np.testing.assert_allclose(loss[0], lo, rtol=1e-13, atol=0)
        np.testing.assert_allclose(grad[0], go, rtol=1e-13, atol=1e-300)


@pytest.mark.parametrize("n", [1, 2, 11, 12, 13, 14, 31])
def test_live_adjoints(nd, oracle_mod, n):
    """Fewer, as many and more adjoints alive at a time than the reverse sweep
    holds in LDS (the others go through the wave's slot)."""
    bc = held_values(n)
    p = np.random.default_rng(n).uniform(-1.0, 1.0, (70, 2))
    lo, go, _ = oracle_mod.run(bc, p, [])
    loss, grad = walk(nd, [bc], p[None], [])
    np.testing.assert_allclose(loss[0], lo, rtol=1e-13, atol=1e-15 * n)
    np.testing.assert_allclose(grad[0], go, rtol=1e-12, atol=1e-13 * n)


@pytest.mark.parametrize("op", [B.MUL, B.SUB])
def test_record_chunks(nd, oracle_mod, op):
    """Operation counts around the chunks of 64 records and the distance the
    values are read ahead, several programs a launch."""
    counts = [1, 2, 3, 4, 5, 63, 64, 65, 66, 67, 127, 128, 129, 200]
    p = np.random.default_rng(3).uniform(0.9, 1.1, (len(counts), 65, 2))
    codes = [chain(op, n) for n in counts]
    loss, grad = walk(nd, codes, p, [])
    for q, c in enumerate(codes):
        lo, go, _ = oracle_mod.run(c, p[q], [])
        np.testing.assert_allclose(loss[q], lo, rtol=1e-13, atol=1e-13)
        np.testing.assert_allclose(grad[q], go, rtol=1e-13, atol=1e-13)


def test_argument_errors(nd):
    bc = Asm(2, 3).param(0).obs(0).mul().param(1).add().halt().bytes()
    with pytest.raises(nd.NdvmError) as e:
        nd.walk_prepare([configs.kalman(L=2, T=2).bytecode])
    assert e.value.status == nd.E_UNSUPPORTED
    with pytest.raises(nd.NdvmError) as e:
        nd.walk_prepare([bc, Asm(1, 2).param(0).halt().bytes()])
    assert e.value.status == nd.E_ARG          # differing observation counts
    ws = nd.walk_prepare([bc])
    L = 70
    p = torch.ones((L, 2), dtype=torch.float64, device="cuda")
    o = torch.ones(3, dtype=torch.float64, device="cuda")
    loss = torch.full((L,), 5.5, dtype=torch.float64, device="cuda")
    g = torch.full((L, 2), 5.5, dtype=torch.float64, device="cuda")
    need = nd.walk_workspace_bytes(ws, L)
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    base = [ws.handle, p.data_ptr(), L, 2, L * 2, o.data_ptr(), 3, loss.data_ptr(), g.data_ptr(), 2, L * 2,
            work.data_ptr(), need, s]

    def call(**kw):
        a = list(base)
        for k, v in kw.items():
            a[int(k[1:])] = v
        return nd._walk_grad(*a)

    for what, kw, want in [("null set", dict(a0=None), nd.E_ARG), ("null params", dict(a1=None), nd.E_ARG),
                           ("negative L", dict(a2=-1), nd.E_ARG), ("ld_p < P", dict(a3=1), nd.E_ARG),
                           ("n_obs mismatch", dict(a6=2), nd.E_ARG), ("null loss", dict(a7=None), nd.E_ARG),
                           ("ld_g < P", dict(a9=1), nd.E_ARG),
                           ("workspace too small", dict(a12=need - 8), nd.E_NOMEM)]:
        st = call(**kw)
        assert st == want, (what, st, nd.last_error())
    torch.cuda.synchronize()
    assert torch.all(loss == 5.5) and torch.all(g == 5.5)
    assert call() == nd.OK
    assert call(a2=0) == nd.OK
    nd.walk_status(work)
    torch.cuda.synchronize()
    assert torch.allclose(loss, torch.full_like(loss, 2.0))
    assert torch.allclose(g[:, 0], torch.ones(L, dtype=torch.float64, device="cuda"))


def test_random_program_population_full_size(nd, oracle_mod):
    """The 1,024-program population at its benchmark size (1,024 lanes each)
    in one launch; every program compared with the oracle on lanes 0, 1, 63,
    64, the last and 8 random ones."""
    w = configs.random_programs()
    loss, grad = walk(nd, w.programs, w.params, w.obs)
    rng = np.random.default_rng(2)
    tot = dict(n_lanes=0, n_strict=0, n_ill_conditioned=0, n_libm_sensitive=0, n_other_arm=0)
    for q, bc in enumerate(w.programs):
        P = w.n_params_each[q]
        lanes = np.array(sorted({0, 1, 63, 64, w.L - 1} | set(rng.choice(w.L, 8, replace=False).tolist())))
        r = judge(oracle_mod, bc, w.params[q][lanes][:, :P], w.obs, loss[q, lanes], grad[q, lanes, :P])
        for k in tot:
            tot[k] += r[k]
    record("walk_random_programs_full_size", n_programs=len(w.programs), L=w.L, **tot)
    assert tot["n_other_arm"] <= tot["n_lanes"] // 50
