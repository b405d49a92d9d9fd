"""Captured graphs: every compute call recorded on a stream and replayed several
times, with eager work, new inputs and synchronisations between the replays;
each replay gives the eager call's bits."""
import numpy as np
import pytest

from wide_cases import scalars_and_a_product
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_03574_amd as m
    return m


def replays(call, inputs, outputs, fresh):
    """Capture call() and compare five replays with eager calls.  inputs: tensors
    refilled by fresh(i) before each; outputs: tensors call() writes."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        call(side)                       # outside the capture first, as a program's warm-up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(side)
    for i in range(5):
        for t, v in zip(inputs, fresh(i)):
            t.copy_(v)
        call(torch.cuda.current_stream())
        want = [t.clone() for t in outputs]
        for t in outputs:
            t.fill_(-7.25)
        noise = torch.randn(1 << 20, device="cuda").sum()      # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert noise.isfinite()
        for a, b in zip(outputs, want):
            assert torch.equal(a, b), i


def rows(L, base, seed):
    def fresh(i):
        rng = np.random.default_rng(seed + i)
        return [torch.tensor(base * rng.uniform(0.9, 1.1, (L, base.size)), device="cuda")]
    return fresh


# a scalar program and one with matrices on the wide kernel, small matrices on the slot kernel
PROGRAMS = {"logistic": lambda: (lambda w: (w.bytecode, w.params[0], w.obs))(configs.logistic(L=1, T=40)),
            "kalman": lambda: (lambda w: (w.bytecode, w.params[0], w.obs))(configs.kalman(L=1, T=12)),
            "small": lambda: (scalars_and_a_product(12, 2, 1), np.array([0.21, 0.24, 0.27, 0.3]), np.zeros(1))}


@pytest.mark.parametrize("policy", [1, 2])
@pytest.mark.parametrize("name", sorted(PROGRAMS))
def test_gradients_and_losses(nd, name, policy):
    code, base, obs = PROGRAMS[name]()
    L = 333
    tape = nd.tape_upload(nd.tape_build(code), policy)
    p, o = torch.empty(L, base.size, dtype=torch.float64, device="cuda"), torch.tensor(obs, device="cuda")
    fresh = rows(L, base, 11)
    p.copy_(fresh(0)[0])
    loss, l2, f = (torch.empty(L, dtype=torch.float64, device="cuda") for _ in range(3))
    grad, g2 = torch.empty_like(p), torch.empty_like(p)
    ws = torch.empty(max(nd.workspace_bytes(tape, L, True), nd.workspace_bytes(tape, L, False)), dtype=torch.uint8,
                     device="cuda")

    def call(stream):
        nd.grad(tape, p, o, loss=loss, grad_out=grad, workspace=ws, stream=stream)
        nd.forward(tape, p, o, loss=f, workspace=ws, stream=stream)
        nd.grad_noalloc(tape, p, o, l2, g2, stream=stream)
    replays(call, [p], [loss, grad, f, l2, g2], fresh)
    assert torch.equal(loss, l2) and torch.equal(grad, g2)


def test_walks(nd):
    """The walker, whose status word every call clears: it reads clear after each
    replay, whatever stood there before."""
    w = configs.random_programs(n_prog=6, L=1, n=8, seed=3)
    L, P = 100, w.params.shape[2]
    ws = nd.walk_prepare(w.programs)
    p, o = torch.empty(6, L, P, dtype=torch.float64, device="cuda"), torch.tensor(w.obs, device="cuda")

    def fresh(i):
        return [torch.tensor(np.random.default_rng(i).uniform(-2, 2, (6, L, P)), device="cuda")]
    p.copy_(fresh(0)[0])
    work = torch.empty(nd.walk_workspace_bytes(ws, L), dtype=torch.uint8, device="cuda")
    loss, grad = torch.empty(6, L, dtype=torch.float64, device="cuda"), torch.zeros(6, L, P, dtype=torch.float64, device="cuda")
    status = work[:4].view(torch.int32)
    seen, own = torch.empty(1, dtype=torch.int32, device="cuda"), torch.empty_like(grad)
    written = torch.tensor([[[float(i < n) for i in range(P)]] for n in w.n_params_each], dtype=torch.float64, device="cuda")

    def call(stream):
        with torch.cuda.stream(stream):
            status.fill_(77)
            nd.walk_grad(ws, p, o, loss=loss, grad_out=grad, workspace=work, stream=stream)
            seen.copy_(status)
            torch.mul(grad, written, out=own)
    replays(call, [p], [loss, own, seen], fresh)
    assert seen.item() == 0
    nd.walk_status(work)

