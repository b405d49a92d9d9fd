"""Programs at the edges of the wide replay kernel's blocks, load slots
register file and matrix functions: shared by the emulator and GPU tests."""
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


def large(A):
    """The program with as many 4x4 products appended as make its matrix
    operations large enough for the wide kernel (their result enters the loss)."""
    for i in range(16):
        A.push((0.3, 1.1, 0.3)[i % 3])
    A.pack(4, 4).storel(30).loadl(30).storel(31).loop(8).loadl(31).loadl(30).matmul().storel(31).endloop()
    return A.loadl(31).index(1, 2).mul().halt().bytes()


def long_recurrence(steps):
    """x <- p0 x (1 - x), steps times (three values a rule reads each)."""
    return Asm(2, 0).param(1).storel(0).loop(steps).loadl(0).push(1.0).loadl(0).sub().mul().param(0).mul().storel(0) \
        .endloop().loadl(0).halt().bytes()


def scalars_and_a_product(steps, side, n):
    """A step: a product of side x side matrices, scaled, and n scalar updates."""
    A = Asm(4, 1)
    for i in range(side * side):
        A.param(i % 4)
    A.pack(side, side).storel(0).param(0).storel(2).param(1).storel(3).loadl(0).storel(5).loop(steps)
    A.loadl(0).loadl(5).matmul().param(3).mul().storel(5)
    for _ in range(n):
        A.loadl(2).param(2).mul().loadl(3).add().param(3).mul().storel(2)
    return A.endloop().loadl(5).index(0, 0).loadl(2).add().halt().bytes()


def sum_of_terms(ops, n):
    """Sum over n points of (op(... op(p0 x + p1)) - y)^2: independent chains of
    library functions ("pow" to the power p2, "div" by p3, "mul" by p3)."""
    A = Asm(4, 2 * n).push(0.0).storel(0).loop(n)
    A.param(0).obs(0, 1).mul().param(1).add()
    for op in ops.split():
        if op in ("pow", "div", "mul"):
            A.param(2 if op == "pow" else 3)
        getattr(A, op)()
    return A.obs(n, 1).sub().dup().mul().loadl(0).add().storel(0).endloop().loadl(0).halt().bytes()


def points_of_terms(n):
    return np.concatenate([np.linspace(0.1, 1.0, n), np.linspace(0.2, 0.9, n)])


def network(units, n):
    """Squared residuals of a hidden layer over n points: 3 units + 1 parameters,
    of whose adjoints the register file of the wide kernel has little room left."""
    A = Asm(3 * units + 1, 2 * n).push(0.0).storel(0).loop(n).param(3 * units).storel(1)
    for h in range(units):
        A.push(1.0).obs(0, 1).param(h).mul().param(units + h).add().exp().push(1.0).add().div()
        A.param(2 * units + h).mul().loadl(1).add().storel(1)
    return A.loadl(1).obs(n, 1).sub().dup().mul().loadl(0).add().storel(0).endloop().loadl(0).halt().bytes()


def extended_filter(steps, n, m):
    """An extended Kalman filter's loss: n states, each a sine of its neighbour
    away from the last, m of them observed one after another; transitions and
    Jacobians packed from scalars each step."""
    A = Asm(6, steps * m)
    for p in (4, 5):      # the first covariance, the process noise
        for i in range(n * n):
            A.param(p) if i % (n + 1) == 0 else A.push(0.0)
        A.pack(n, n).storel(6 + p)
    for i in range(n):
        A.param(i % 4)
    A.pack(n, 1).storel(12).push(0.0).storel(20).loop(steps)
    for i in range(n):
        A.loadl(12).index(i, 0).storel(i)
    for i in range(n):
        A.loadl(i).loadl((i + 1) % n).sin().param(3).mul().add()
    A.pack(n, 1).storel(12)
    for i in range(n):
        for j in range(n):
            if j == i:
                A.push(1.0)
            elif j == (i + 1) % n:
                A.loadl(j).cos().param(3).mul()
            else:
                A.push(0.0)
    A.pack(n, n).storel(13).loadl(13).loadl(10).matmul().loadl(13).transpose().matmul().loadl(11).add().storel(10)
    for q in range(m):
        A.obs(q, m).loadl(12).index(q, 0).sub().storel(21).loadl(10).index(q, q).param(4).add().storel(22)
        A.loadl(21).loadl(22).div().storel(23)
        for i in range(n):
            A.loadl(10).index(i, q)
        A.pack(n, 1).loadl(23).mul().loadl(12).add().storel(12)
        A.loadl(21).dup().mul().loadl(22).div().loadl(22).log().add().loadl(20).add().storel(20)
    return A.endloop().loadl(20).halt().bytes()


def lookup(params, n):
    """(p0 * table - y)^2, the table nested branches of n constant leaves over
    thresholds of the other parameters: parameters and constants (which the
    register file holds throughout) and hardly any values."""
    A = Asm(params, 1).param(0)
    for i in range(n):
        A.param(i % (params - 1) + 1).push(0.25 + 0.5 * i).iflt().push(1.0 + i).else_()
    A.push(-1.0)
    for i in range(n):
        A.endif()
    return A.mul().obs(0).sub().dup().mul().halt().bytes()


def lookups():
    """(name, bytecode, observations, parameter rows, whether the file holds
    its parameters, their adjoints and the constants)."""
    rng = np.random.default_rng(23)
    return [(f"lookup{p}_{n}", lookup(p, n), np.ones(1), rng.normal(size=(3, p)), fits)
            for p, n, fits in ((32, 20, False), (28, 30, False), (24, 30, False), (8, 60, False), (32, 8, False),
                               (31, 1, True), (28, 5, True), (8, 20, True), (2, 31, True))]


def one_element_forms():
    """(name, bytecode, observations, parameter rows): matrix words on scalars in
    programs without a matrix, as values, leaves and the loss."""
    rows = np.array([[2.0, 3.0], [-0.0, 1.5], [np.inf, 0.0]])

    def forms(name, apply):
        yield name, apply(Asm(2, 0).param(0)).param(1).mul()
        yield name + "_loss", apply(Asm(2, 0).param(0).param(1).mul())
        yield name + "_const", apply(Asm(2, 0).push(0.75)).param(1).mul().param(0).sub()
        yield name + "_shared", apply(Asm(2, 0).param(0).param(1).sub().dup()).mul().dup().add()
        A = Asm(2, 2).param(0).storel(0).loop(20)      # several segments, observations
        yield name + "_loop", apply(A.loadl(0).param(1).mul().sin()).dup().storel(0).obs(1).sub().storel(1) \
            .endloop().loadl(1).loadl(0).add()
    out = []
    for name, apply in (("pack1", lambda A: A.pack(1, 1)), ("index1", lambda A: A.index(0, 0)),
                        ("transpose1", lambda A: A.transpose())):
        out += [(n, A.halt().bytes(), np.array([0.5, -1.25] if n.endswith("loop") else []), rows) for n, A in forms(name, apply)]
    return out


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
    # matrices: every shape of a product and of its adjoints, both operands and
    # results of one element, transposes, differences, packs of repeated and
    # constant elements, elements taken out, inverses and log-determinants
    for m in (1, 2, 3, 4):
        for k in (1, 2, 3, 4):
            for n in (1, 2, 3, 4):
                A = Asm(m * k + k * n, 0)
                for i in range(m * k):
                    A.param(i)
                A.pack(m, k)
                for i in range(k * n):
                    A.param(m * k + i)
                A.pack(k, n).matmul().storel(0).push(0.0)
                for i in range(m):
                    for j in range(n):
                        A.loadl(0).index(i, j).push((0.3, -0.7, 1.1)[(i + 2 * j) % 3]).mul().add()
                if m * k + k * n <= 16:      # the register file holds the parameters and their adjoints
                    add(f"matmul{m}{k}{n}", large(A), [], rng.normal(size=(2, m * k + k * n)))
    A = Asm(6, 2)
    for i in (0, 1, 2, 3, 4, 5):
        A.param(i)
    A.pack(2, 3).storel(0).param(0).param(0).push(1.5).obs(0).obs(1).param(5).pack(3, 2).storel(1)
    A.loadl(0).loadl(1).transpose().sub().storel(2).loadl(2).loadl(2).transpose().matmul().storel(3)
    A.param(1).loadl(3).mul().param(2).mul().loadl(3).add().storel(4).loadl(4).inv().storel(5)
    A.loadl(5).loadl(3).matmul().logdet().loadl(5).index(0, 1).mul().loadl(4).logdet().add().loadl(2).index(1, 2).add()
    add("matrices", large(A), [0.5, -1.25], rng.normal(size=(5, 6)))
    A = Asm(5, 0)      # a node whose adjoint is zero against infinite operands
    for i in range(4):
        A.param(i)
    A.pack(2, 2).dup().matmul().storel(0).loadl(0).loadl(0).transpose().matmul().index(0, 0).param(4).mul()
    add("matrix_zero_inf", large(A), [], [[np.inf, 1.0, 2.0, 3.0, 0.0], [1.0, -0.0, 2.0, 3.0, 0.0],
                                                  [1e200, 1e200, 1.0, 1.0, 1.0], [0.5, 0.25, -1.0, 2.0, 1.0]])
    for T in (1, 2, 5):
        w = configs.kalman(L=3, T=T)
        add(f"kalman{T}", w.bytecode, w.obs, w.params)
    for seed in range(6):
        w = configs.random_programs(n_prog=3, L=4, n=9, seed=900 + seed)
        for q, code in enumerate(w.programs):
            add(f"tree{seed}_{q}", code, w.obs, w.params[q, :, : w.n_params_each[q]])
    return out
