"""Scalar programs at the edges of the wide replay kernel's blocks, load slots
and register file: shared by the emulator and GPU tests."""
import numpy as np

from workloads import configs
from workloads import bytecode as B
from workloads.bytecode import Asm


def chain(op, n, params=2):
    """x <- x op p1 n times (runs of one class: full blocks and remainders)."""
    A = Asm(params, 0).param(0).storel(0)
    for _ in range(n):
        A.loadl(0).param(1).raw(op).storel(0)
    return A.loadl(0).halt().bytes()


def unary_chain(op, n):
    A = Asm(1, 0).param(0)
    for _ in range(n):
        A.raw(op)
    return A.halt().bytes()


def sum_of_obs(n, scale):
    """sum over n observations of (p0 - y)^2 * scale (load batches and their halves)."""
    A = Asm(1, n).push(0.0).storel(0).loop(n)
    A.loadl(0).param(0).obs(0, 1).sub().dup().mul().push(scale).mul().add().storel(0).endloop()
    return A.loadl(0).halt().bytes()


def held_values(n):
    """n values formed first and read last (registers, then more checkpoint
    segments than one)."""
    A = Asm(2, 0).param(0).storel(n)
    for i in range(n):
        A.loadl(n).param(1).add().sin().dup().storel(n).storel(i)
    A.push(0.0)
    for i in range(n):
        A.loadl(i).loadl(n - 1 - i).mul().add()
    return A.halt().bytes()


def branch(then_first):
    """Nested selects whose arms are parameters, values and constants."""
    A = Asm(3, 0).param(0).param(1).iflt()
    A.param(2).param(0).mul().else_()
    A.param(0).param(1).iflt().push(2.0).else_().param(1).exp().endif()
    A.endif()
    if then_first:
        A.param(0).param(0).iflt().param(1).else_().param(2).endif().add()
    return A.dup().mul().halt().bytes()


def cases():
    """(name, bytecode, observations, parameter rows)."""
    rng = np.random.default_rng(17)
    out = []

    def add(name, code, obs, rows):
        out.append((name, code, np.asarray(obs, dtype=np.float64), np.asarray(rows, dtype=np.float64)))

    for op, name in ((B.ADD, "add"), (B.SUB, "sub"), (B.MUL, "mul"), (B.DIV, "div")):
        for n in (1, 4, 5, 8, 9, 10, 11, 15, 16, 31):
            add(f"{name}{n}", chain(op, n), [], rng.uniform(0.7, 1.3, (3, 2)))
    for op, name in ((B.EXP, "exp"), (B.LOG, "log"), (B.SQRT, "sqrt"), (B.SIN, "sin"), (B.COS, "cos"), (B.ABS, "abs"),
                     (B.NEG, "neg")):
        for n in (1, 2, 11):
            x = rng.uniform(0.2, 0.9, (3, 1)) * (0.1 if op == B.EXP else 1.0)
            if op == B.LOG:
                x = np.array([[1e-9], [3.0], [20.0]])
            add(f"{name}{n}", unary_chain(op, n), [], x)
    add("pow3", chain(B.POW, 3), [], rng.uniform(0.8, 1.2, (3, 2)))
    for n in (1, 3, 4, 5, 8, 9, 13, 17):
        add(f"obs{n}", sum_of_obs(n, 1.0 / n), rng.normal(size=n), rng.normal(size=(3, 1)))
    for n in (3, 20, 40, 60):
        add(f"held{n}", held_values(n), [], rng.uniform(-1.0, 1.0, (3, 2)))
    for f in (False, True):
        add(f"branch{int(f)}", branch(f), [],
            [[1.0, 2.0, 3.0], [2.0, 1.0, 3.0], [1.0, 1.0, -2.0], [np.nan, 1.0, 2.0], [3.0, 800.0, 0.5]])
    # zero adjoints against infinite operands, overflow, the loss a parameter, a constant, an observation
    add("zero_times_inf", Asm(3, 0).param(0).param(1).mul().param(2).mul().halt().bytes(), [],
        [[np.inf, 1.0, 0.0], [0.0, np.inf, 2.0], [1e200, 1e200, 0.0], [-0.0, 3.0, 1.0]])
    add("zero_over", Asm(3, 0).param(0).param(1).div().param(2).mul().halt().bytes(), [],
        [[1.0, 0.0, 0.0], [0.0, 0.0, 1.0], [1.0, np.inf, 0.0], [5e-324, 1e-300, 1.0]])
    add("loss_param", Asm(2, 0).param(1).halt().bytes(), [], [[1.0, -2.5]])
    add("loss_const", Asm(1, 0).push(3.25).halt().bytes(), [], [[1.0]])
    add("loss_obs", Asm(1, 2).obs(1).halt().bytes(), [4.0, 5.5], [[1.0]])
    add("no_params", Asm(0, 1).obs(0).exp().halt().bytes(), [0.5], np.zeros((2, 0)))
    add("square", Asm(1, 0).param(0).dup().mul().dup().mul().halt().bytes(), [], [[1.5], [-0.0]])
    w = configs.exp_decay(L=3, n=21)
    add("exp_decay", w.bytecode, w.obs, w.params)
    w = configs.logistic(L=3, T=37)
    add("logistic", w.bytecode, w.obs, w.params)
    for T in (1, 2, 60):
        w = configs.lotka_volterra(L=3, T=T)
        add(f"lotka{T}", w.bytecode, w.obs, w.params)
    for seed in range(6):
        w = configs.random_programs(n_prog=3, L=4, n=9, seed=900 + seed)
        for q, code in enumerate(w.programs):
            add(f"tree{seed}_{q}", code, w.obs, w.params[q, :, : w.n_params_each[q]])
    return out
