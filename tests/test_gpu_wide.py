"""Wide replay kernel on the GPU: every case at the edges of its format against
the oracle (both policies, forward, ragged lane counts), and the static-scratch
entry point in parts."""
import numpy as np
import pytest

from parity import compare
from wide_cases import cases, long_recurrence, scalars_and_a_product
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_03574_amd as m
    return m


@pytest.mark.parametrize("L", [1, 65])
def test_cases_equal_oracle(nd, oracle_mod, L):
    for name, code, obs, rows in cases():
        if rows.shape[1] == 0:     # the binding takes no empty parameter rows
            continue
        p = np.ascontiguousarray(rows[np.arange(L) % len(rows)])
        ol, og, _ = oracle_mod.run(code, p, obs)
        t = nd.tape_build(code)
        P, O = torch.tensor(p, device="cuda"), torch.tensor(obs, device="cuda")
        for policy in (nd.POLICY_RECOMPUTE, nd.POLICY_SAVE):
            print(name, L, policy, flush=True)
            tape = nd.tape_upload(t, policy)
            loss, grad = nd.grad(tape, P, O)
            f = nd.forward(tape, P, O)
            torch.cuda.synchronize()
            assert torch.equal(f.isnan(), loss.isnan()) and torch.equal(f.nan_to_num(), loss.nan_to_num()), name
            grads = (grad.cpu().numpy(), og) if og.size else (None, None)
            compare(loss.cpu().numpy(), grads[0], ol, grads[1])


def test_cases_of_many_waves(nd):
    """The same cases on as many lanes as leave them to the wide kernel, whatever
    their operations: the bits of the small launches, in every copy of a row."""
    L = 16 * 4 * 256 + 65
    for name, code, obs, rows in cases():
        if rows.shape[1] == 0:
            continue
        few = rows[np.arange(65) % len(rows)]
        P, p, O = (torch.tensor(np.ascontiguousarray(x), device="cuda") for x in (rows[np.arange(L) % len(rows)], few, obs))
        t = nd.tape_build(code)
        for policy in (nd.POLICY_RECOMPUTE, nd.POLICY_SAVE):
            print(name, policy, flush=True)
            tape = nd.tape_upload(t, policy)
            big, small = [*nd.grad(tape, P, O), nd.forward(tape, P, O)], [*nd.grad(tape, p, O), nd.forward(tape, p, O)]
            torch.cuda.synchronize()
            for a, b in zip(big, small):
                b = b[:len(rows)].repeat([-(-L // len(rows))] + [1] * (b.dim() - 1))[:L]
                assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num()), name


def test_noalloc_in_parts_equals_grad(nd):
    """A scalar launch whose rows exceed the static scratch array runs in parts
    of its lanes (the last one ragged), with the results of one launch."""
    w = configs.lotka_volterra(L=13007, T=1000)
    tape = nd.tape_upload(nd.tape_build(w.bytecode))
    p, o = torch.tensor(w.params, device="cuda"), torch.tensor(w.obs, device="cuda")
    assert nd.workspace_bytes(tape, 13007, True) > nd.NOALLOC_SCRATCH_BYTES
    l0, g0 = nd.grad(tape, p, o)
    l1, g1 = torch.empty_like(l0), torch.empty_like(g0)
    nd.grad_noalloc(tape, p, o, l1, g1)
    torch.cuda.synchronize()
    assert torch.equal(l0, l1) and torch.equal(g0, g1)


@pytest.mark.parametrize("name,L,steps", [("kalman", 2003, 60), ("mixed", 8000, 200)])
def test_noalloc_of_matrix_programs_in_parts(nd, name, L, steps):
    """Programs with matrices that need two and six times the scratch array, the
    last part ragged; beyond four only because the program recomputes from few
    values (the Kalman filter that saves is refused there)."""
    if name == "kalman":
        w = configs.kalman(L=L, T=steps)
        code, p, obs, policy = w.bytecode, w.params, w.obs, nd.POLICY_SAVE
    else:
        code, obs, policy = scalars_and_a_product(steps, 4, 30), np.zeros(1), nd.POLICY_RECOMPUTE
        p = np.random.default_rng(3).uniform(0.2, 0.3, (L, 4))
    tape = nd.tape_upload(nd.tape_build(code), policy)
    P, O = torch.tensor(p, device="cuda"), torch.tensor(obs, device="cuda")
    need = nd.workspace_bytes(tape, L, True) / nd.NOALLOC_SCRATCH_BYTES
    assert (1.5 < need < 4) if name == "kalman" else (4 < need < 8)
    l0, g0 = nd.grad(tape, P, O)
    l1, g1 = torch.empty_like(l0), torch.empty_like(g0)
    nd.grad_noalloc(tape, P, O, l1, g1)
    torch.cuda.synchronize()
    assert torch.equal(l0, l1) and torch.equal(g0, g1) and not g0.isnan().any()
    if name == "kalman":
        P = P.repeat(4, 1)
        assert nd.workspace_bytes(tape, 4 * L, True) > 4 * nd.NOALLOC_SCRATCH_BYTES
        l1, g1 = torch.full((4 * L,), -7.25, dtype=torch.float64, device="cuda"), torch.empty_like(P)
        with pytest.raises(nd.NdvmError) as e:
            nd.grad_noalloc(tape, P, O, l1, g1)
        assert e.value.status == nd.E_NOMEM and "static scratch" in str(e.value)
        torch.cuda.synchronize()
        assert torch.all(l1 == -7.25)


def test_more_rows_than_the_scratch_array_holds(nd, oracle_mod):
    """A saving program of which one wave exceeds the static scratch array: the
    wide kernel runs it on a caller's workspace, alone and in a population
    (its rows, fewer than the slot program's), and the array is too small."""
    import emu
    code = long_recurrence(90000)
    t = nd.tape_build(code)
    rows = emu.wide(t, np.zeros((0, 2)), np.zeros(0), 2)[2]["n_ckpt_rows"] + 4
    p = np.array([[2.6, 0.3], [2.9, 0.6], [1.5, 0.9]])
    L = 70
    p = np.ascontiguousarray(p[np.arange(L) % 3])
    ol, og, _ = oracle_mod.run(code, p, np.zeros(0))
    P, O = torch.tensor(p, device="cuda"), torch.zeros(0, dtype=torch.float64, device="cuda")
    tape = nd.tape_upload(t, nd.POLICY_SAVE)
    assert nd.workspace_bytes(tape, L, True) == rows * 128 * 8 > nd.NOALLOC_SCRATCH_BYTES
    assert nd.workspace_bytes_many([tape], L) == rows * 128 * 8
    loss, grad = nd.grad(tape, P, O)
    torch.cuda.synchronize()
    compare(loss.cpu().numpy(), grad.cpu().numpy(), ol, og)
    with pytest.raises(nd.NdvmError) as e:
        nd.grad_noalloc(tape, P, O, loss, grad)
    assert e.value.status == nd.E_NOMEM and "static scratch" in str(e.value)
