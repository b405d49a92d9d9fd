"""Which kernel serves a call, on the GPU against the oracle: populations and
data-axis launches of programs with matrices, populations that mix them with
scalar programs, terms and programs that only the slot kernel takes, and the
wide kernel with half the LDS a wave."""
import numpy as np
import pytest

import emu
from parity import compare, judge
from test_gpu_points import check
from wide_cases import (branch, extended_filter, lookups, network, one_element_forms, points_of_terms,
                        scalars_and_a_product, sum_of_terms)
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


def dev(x):
    return torch.tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


def many(nd, oracle_mod, codes, L, policy, seed=1):
    """grad_many of programs of four parameters and one observation, each against
    the oracle and against its own launch; returns the tapes."""
    tapes = [nd.tape_upload(t, policy) for t in (nd.tape_build(c) for c in codes)]
    p = np.random.default_rng(seed).uniform(0.2, 0.3, (len(codes), L, 4))
    obs = np.array([0.4])
    loss, grad = nd.grad_many(tapes, dev(p), dev(obs))
    torch.cuda.synchronize()
    for q, code in enumerate(codes):
        ol, og, _ = oracle_mod.run(code, p[q], obs)
        compare(loss[q].cpu().numpy(), grad[q].cpu().numpy(), ol, og)
        l1, g1 = nd.grad(tapes[q], dev(p[q]), dev(obs))
        assert torch.equal(l1, loss[q]) and torch.equal(g1, grad[q]), q
    return tapes


KINDS = [(1, 4, 0), (3, 3, 0), (7, 4, 2), (12, 3, 1), (20, 4, 0)]   # steps, side, scalar updates
MATRIX = [scalars_and_a_product(*k) for k in KINDS]


@pytest.mark.parametrize("policy", [1, 2])
@pytest.mark.parametrize("L", [1, 77])
def test_population_of_matrix_programs(nd, oracle_mod, L, policy):
    """Forty programs of five LDS sizes (laid out per XCD), and three (on the
    grid's second axis): the program table's rows, the launch's LDS, blocks of
    16 lanes with a ragged last one."""
    mode = 2 if policy == nd.POLICY_SAVE else 1
    stats = [emu.wide(nd.tape_build(c), np.zeros((0, 4)), np.zeros(1), mode, lds_rows=1280)[2] for c in MATRIX]
    assert all(s["pays"] for s in stats) and len({s["lds_rows"] for s in stats}) > 1
    tapes = many(nd, oracle_mod, MATRIX * 8, L, policy)
    want = sum((s["n_ckpt_rows"] + 4) * 8 for s in stats) * -(-L // 64) * 64 * 8
    assert nd.workspace_bytes_many(tapes, L) == want
    many(nd, oracle_mod, MATRIX[:3], L, policy, seed=2)


def scalar_program():
    A = Asm(4, 1).push(0.0).storel(0).loop(9)
    return A.loadl(0).param(0).param(1).mul().obs(0).sub().sin().add().param(2).mul().storel(0).endloop().loadl(0) \
        .param(3).add().dup().mul().halt().bytes()


def test_population_of_scalar_and_matrix_programs(nd, oracle_mod):
    """One launch of programs that the two wide kernels would take apart: the
    slot kernel's (its workspace, not theirs)."""
    codes = [scalar_program(), MATRIX[2], scalar_program(), MATRIX[3]]
    tapes = many(nd, oracle_mod, codes, 50, nd.POLICY_SAVE)
    alone = sum(nd.workspace_bytes(t, 50, True) for t in tapes)
    slot = sum(emu.run(nd.tape_build(c), np.zeros((0, 4)), np.zeros(1), budget=1280, save=True)[2]["n_ckpt_rows"] + 4
               for c in codes)
    assert nd.workspace_bytes_many(tapes, 50) == slot * 64 * 8 != alone


def matrix_term():
    """(c^T A^2 c - y)^2 of a 4x4 matrix of the parameters and the point."""
    A = Asm(4, 2)
    for i in range(16):
        A.param(i % 4) if i % 3 else A.obs(0)
    A.pack(4, 4).storel(0).param(0).param(1).param(2).obs(0).pack(4, 1).storel(1)
    A.loadl(0).loadl(0).matmul().loadl(0).matmul().storel(2)
    A.loadl(1).transpose().loadl(2).matmul().loadl(1).matmul().obs(1).sub().dup().mul()
    return A.halt().bytes()


@pytest.mark.parametrize("L,N", [(1, 1), (37, 13), (3, 200)])
def test_points_of_a_matrix_term(nd, oracle_mod, L, N):
    term = matrix_term()
    assert emu.wide(nd.tape_build(term), np.zeros((0, 4)), np.zeros(2))[2]["pays"]
    rng = np.random.default_rng(L * N)
    tot = check(nd, oracle_mod, term, rng.uniform(0.5, 1.5, (L, 4)), rng.normal(size=(N, 2)), 1.0 / N)
    assert tot["n_strict"] == L * N


@pytest.mark.parametrize("policy", [1, 2, 1 | 0x100, 2 | 0x100])
def test_points_of_a_term_the_slot_kernel_runs(nd, oracle_mod, policy):
    """A term of more parameters than the wide kernel's file holds, and (with the
    branch-skipping option) one with a branch."""
    from oracle import flatten
    A = Asm(40, 2).obs(0)
    for i in range(40):
        A.param(i).mul().obs(0).add()
    big = A.obs(1).sub().dup().mul().halt().bytes()
    assert emu.wide(nd.tape_build(big), np.zeros((0, 40)), np.zeros(2)) is None
    small = Asm(2, 2).param(0).obs(0).iflt()
    for _ in range(12):
        small.param(1).mul().obs(0).add() if _ else small.param(0).param(1).mul()
    small.else_().param(0).obs(1).sub().sin().endif().dup().mul()
    rng = np.random.default_rng(9)
    for term, P in ((big, 40), (small.halt().bytes(), 2)):
        p, pts = rng.uniform(0.4, 0.9, (21, P)), rng.uniform(0.3, 1.0, (11, 2))
        tape = nd.tape_upload(nd.tape_build(term), policy)
        loss, grad = nd.grad_points(tape, dev(p), dev(pts), 1.0 / 11)
        torch.cuda.synchronize()
        compare(loss.cpu().numpy(), grad.cpu().numpy(), *flatten.run_points(term, p, pts, 1.0 / 11))


@pytest.mark.parametrize("policy", [1, 2])
def test_programs_at_the_register_files_end(nd, oracle_mod, policy):
    """Parameters and constants that fill the wide kernel's file or pass its end,
    and matrix words on scalars."""
    for name, code, obs, rows, *_ in lookups() + one_element_forms():
        p = np.ascontiguousarray(rows[np.arange(67) % len(rows)])
        ol, og, _ = oracle_mod.run(code, p, obs)
        t = nd.tape_build(code)
        for tape in [nd.tape_upload(t, policy)] + nd.tape_upload_many([nd.tape_build(branch(False)), t], policy)[1:]:
            loss, grad = nd.grad(tape, dev(p), dev(obs))
            f = nd.forward(tape, dev(p), dev(obs))
            torch.cuda.synchronize()
            compare(loss.cpu().numpy(), grad.cpu().numpy(), ol, og)
            compare(f.cpu().numpy(), None, ol, None)


def test_half_the_lds_a_wave(nd, oracle_mod):
    """A product of matrices a step on more than six waves a CU: the program made
    for half the LDS (shorter segments), two waves a SIMD."""
    code, L = scalars_and_a_product(8, 4, 0), 6 * 256 * 16 + 25
    t, none = nd.tape_build(code), np.zeros((0, 4))
    full, half = (emu.wide(t, none, np.zeros(1), 1, lds_rows=r)[2] for r in (320, 160))
    assert full["lds_rows"] > 160 >= half["lds_rows"] and half["n_ckpt_rows"] != full["n_ckpt_rows"]
    tape = nd.tape_upload(t)
    padded = -(-L // 64) * 64
    assert nd.workspace_bytes(tape, L, True) == (half["n_ckpt_rows"] + 4) * padded * 8
    assert nd.workspace_bytes(tape, 4096, True) == (emu.wide(t, none, np.zeros(1), 1, lds_rows=1280)[2]["n_ckpt_rows"] + 4) * 4096 * 8
    p = np.random.default_rng(4).uniform(0.2, 0.3, (L, 4))
    loss, grad = nd.grad(tape, dev(p), dev(np.zeros(1)))
    torch.cuda.synchronize()
    ol, og, _ = oracle_mod.run(code, p, np.zeros(1))
    compare(loss.cpu().numpy(), grad.cpu().numpy(), ol, og)


@pytest.mark.parametrize("ops", ["pow pow", "sin sin sin", "extended filter", "network"])
def test_few_waves_of_library_functions(nd, oracle_mod, ops):
    """Losses, and gradients of three sines, of a launch of few waves run on the
    slot kernel; they are the bits of the same lanes in a launch of many, which
    the wide kernel runs, also without a workspace, in a population and with a
    workspace that was sized for gradients only."""
    L, M = 333, 66000
    code, obs, P = {"extended filter": lambda: (extended_filter(24, 4, 2), np.linspace(0.1, 0.9, 48), 6),
                    "network": lambda: (network(8, 40), points_of_terms(40), 25)}.get(
                        ops, lambda: (sum_of_terms(ops, 64), points_of_terms(64), 4))()
    t = nd.tape_build(code)
    rows = np.random.default_rng(6).uniform(0.5, 1.0, (M, P))
    p, o, few = dev(rows), dev(obs), dev(rows[:L])
    tape, other = nd.tape_upload(t), nd.tape_upload_many([t])[0]
    lanes = {n: -(-n // 64) * 64 for n in (L, M)}
    def wide(rows):
        return emu.wide(t, np.zeros((0, P)), obs, 1, lds_rows=rows)[2]["n_ckpt_rows"] + 4
    slot = emu.run(t, np.zeros((0, P)), obs, budget=1280)[2]["n_ckpt_rows"] + 4
    on_slot = emu.route(t, L, 1)[0]
    assert on_slot == (ops != "pow pow") and emu.route(t, L, 0)[0] and slot != wide(1280)
    assert nd.workspace_bytes(tape, L, True) == (slot if on_slot else wide(1280)) * lanes[L] * 8
    assert nd.workspace_bytes(tape, M, True) in [wide(r) * lanes[M] * 8 for r in (320, 160)]
    loss, grad = nd.grad(tape, p, o)
    l0 = nd.forward(tape, p, o)
    l1, g1 = nd.grad(tape, few, o)
    l2 = nd.forward(tape, few, o)
    l3, g3 = torch.empty_like(l1), torch.empty_like(g1)
    nd.grad_noalloc(tape, few, o, l3, g3)
    work = torch.empty(nd.workspace_bytes(other, L, True), dtype=torch.uint8, device="cuda")
    l4 = torch.empty_like(l1)      # (no sizing call for losses: the wide kernel)
    assert nd._forward(other.handle, few.data_ptr(), L, P, o.data_ptr(), o.numel(), l4.data_ptr(), work.data_ptr(),
                       work.numel(), torch.cuda.current_stream().cuda_stream) == nd.OK
    lm, gm = nd.grad_many([tape, other], torch.stack([few, few]), o)
    torch.cuda.synchronize()
    for x in (l1, l2, l3, l4, lm[0], lm[1]):
        assert torch.equal(x, loss[:L])
    assert torch.equal(l0, loss)
    for x in (g1, g3, gm[0], gm[1]):
        assert torch.equal(x, grad[:L])
    # (the filter's sines amplify the last ulps of a math library: the judge's rule)
    judge(oracle_mod, code, rows[:L], obs, l1.cpu().numpy(), g1.cpu().numpy())


def test_points_of_a_term_of_library_functions(nd, oracle_mod):
    """A data-axis launch of few waves whose term the slot kernel runs, and one of
    many lanes."""
    A = Asm(4, 2).param(0).obs(0).mul().param(1).add().sin().sin().sin().sin().sin().sin().obs(1).sub().dup().mul()
    term = A.halt().bytes()
    rng = np.random.default_rng(8)
    for L, N in ((37, 13), (600, 128)):
        tot = check(nd, oracle_mod, term, rng.uniform(0.5, 1.0, (L, 4)), rng.uniform(0.2, 0.9, (N, 2)), 1.0 / N)
        assert tot["n_strict"] == L * N
