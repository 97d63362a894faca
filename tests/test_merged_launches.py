"""Launches that take another region's work along, and the programs where they must not (host logic, null device):
which launches a plan has and what they read and write."""
import numpy as np
import pytest

from paper_2102_13267_amd import Context
from test_launches import check_launches
from test_schedule import hazards_are_ordered, invariants, parse


def schedule(build):
    ctx = Context()

    def mk(shape, dtype="f32", donatable=False):
        return ctx.tensor(np.zeros(shape, np.int32 if dtype == "s32" else np.float32), dtype=dtype, donatable=donatable)
    keep = build(ctx, mk)
    info = ctx.barrier()
    sched = parse(ctx.dump_schedule())
    invariants(sched)
    hazards_are_ordered(sched)
    check_launches(ctx.dump_key(), info.n_nodes, ctx.dump_plan(), sched)
    del keep
    return sched


def kinds(sched):
    return [l["kind"] for l in sched]


# ---- a norm's column reductions behind its input gradient ----------------------------------------------
def norm_gradient(reduce, dt="f32", rows=64, cols=256, between=None):
    """The input gradient, then `reduce` of dy * xhat over the rows."""
    def build(B, mk):
        x, dy = mk((rows, cols), dt, True), mk((rows, cols), dt, True)
        y, mu, rs = B.layer_norm(x, mk((cols,), dt), mk((cols,), dt), eps=1e-5)
        dx = B.layer_norm_grad(dy, x, mk((cols,), dt), mu, rs)
        out = [between(B, x, dy)] if between else []
        xhat = B.mul(B.sub(x, B.reshape(mu, (rows, 1))), B.reshape(rs, (rows, 1)))
        return [y, dx, getattr(B, reduce)(B.mul(dy, xhat), axis=0), x, dy] + out
    return build


def column_operands(sched):
    """How many tensors the column launch reads."""
    (col,) = [l for l in sched if l["kind"] == "COL"]
    return len(col["reads"])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("reduce,operands", [("sum", 1), ("mean", 1), ("amax", 4)])
def test_sums_and_means_ride_with_a_norms_gradient(dt, reduce, operands):
    """(one operand: the partial sums that the gradient's launch has left)"""
    assert column_operands(schedule(norm_gradient(reduce, dt))) == operands


@pytest.mark.parametrize("which", ["x", "dy"])
def test_sums_of_an_overwritten_operand_keep_their_launch(which):
    """The sums are of the operand's new value, which the gradient's launch does not read."""
    def build(B, mk):
        x, dy = mk((64, 256), "f32", True), mk((64, 256), "f32", True)
        y, mu, rs = B.layer_norm(x, mk((256,)), mk((256,)), eps=1e-5)
        dx = B.layer_norm_grad(dy, x, mk((256,)), mu, rs)
        t = x if which == "x" else dy
        B.assign(t, B.mul(t, 0.5))
        return [y, dx, B.sum(B.mul(dy, B.mul(B.sub(x, B.reshape(mu, (64, 1))), B.reshape(rs, (64, 1)))), axis=0), x, dy]
    assert column_operands(schedule(build)) == 4


@pytest.mark.parametrize("dt,rows,cols,operands", [("bf16", 64, 2048, 1), ("bf16", 64, 2056, 4), ("bf16", 64, 252, 4), ("f32", 64, 1024, 1), ("f32", 64, 1028, 4)])
def test_rows_whose_sums_ride(dt, rows, cols, operands):
    """Whole 16-byte chunks, at most four to a lane."""
    assert column_operands(schedule(norm_gradient("sum", dt, rows, cols))) == operands


def test_sums_of_two_norms():
    """Each with the gradient that reads its operands; the same sum twice rides once."""
    def build(B, mk):
        out = []
        for _ in range(2):
            out += norm_gradient("sum")(B, mk)
        return out
    sched = schedule(build)
    assert [len(l["reads"]) for l in sched if l["kind"] == "COL"] == [1, 1]
    written = [l["writes"] for l in sched if l["kind"] == "ROWOP"]
    for col in (l for l in sched if l["kind"] == "COL"):
        assert sum(col["reads"] <= w for w in written) == 1


# ---- a cross-entropy, its gradient and the sum of the losses --------------------------------------------
def losses(B, mk, rows=64, cols=100, order="loss first", reduce="mean", other=False, into=None):
    z, labels = mk((rows, cols), "f32", into == "logits"), mk((rows,), "s32")
    second = mk((rows,), "s32") if other else labels
    if order == "loss first":
        loss, d = B.xent(z, labels), B.xent_grad(z, second, 0.5)
    else:
        d = B.xent_grad(z, labels, 0.5)
        loss = B.xent(z, second)
    if into:
        w = z if into == "logits" else mk((rows, cols), "f32", True)
        B.assign(w, d)
        d = w
    return [d, getattr(B, reduce)(loss) if reduce else loss]


@pytest.mark.parametrize("order", ["loss first", "gradient first"])
def test_a_loss_its_gradient_and_their_mean_are_one_launch(order):
    for reduce in ("mean", "sum", None):
        assert kinds(schedule(lambda B, mk: losses(B, mk, order=order, reduce=reduce))) == ["ROWOP"]


@pytest.mark.parametrize("order", ["loss first", "gradient first"])
def test_a_gradient_of_other_labels_has_its_own_launch(order):
    sched = schedule(lambda B, mk: losses(B, mk, order=order, other=True))
    assert kinds(sched) == ["ROWOP", "ROWOP"]


def test_a_gradient_written_into_a_parameter():
    """Not before its place, where another launch may still read the old value: behind the loss, in a launch of its own.  (Its
    own logits it never overwrites, so those two share a launch.)"""
    def build(B, mk):
        w = mk((64, 100), "f32", True)
        z, labels = mk((64, 100)), mk((64,), "s32")
        loss, old = B.xent(z, labels), B.sum(w, axis=1)
        B.assign(w, B.xent_grad(z, labels, 0.5))
        return [loss, old, w]
    sched = schedule(build)
    assert kinds(sched).count("ROWOP") == 2
    (over,) = [l for l in sched if any(w.startswith("p") for w in l["writes"])]
    assert all(l["i"] < over["i"] for l in sched if l["reads"] & over["writes"]) and len(over["writes"]) == 1
    assert kinds(schedule(lambda B, mk: losses(B, mk, into="logits"))) == ["ROWOP"]


def test_other_reductions_of_the_losses_have_their_own_launch():
    assert kinds(schedule(lambda B, mk: losses(B, mk, reduce="amax"))) == ["ROWOP", "ALL"]

    def squares(B, mk):
        d, loss = losses(B, mk, reduce=None)
        return [d, loss, B.sum(B.square(loss))]
    assert kinds(schedule(squares)) == ["ROWOP", "ALL"]

    def finaliser(B, mk):
        d, loss = losses(B, mk, reduce=None)
        return [d, B.div(loss, B.sum(loss))]
    assert kinds(schedule(finaliser)) == ["ROWOP", "ALL"]

    def running(B, mk):
        d, loss = losses(B, mk, reduce=None)
        s = mk((), "f32", True)
        B.assign(s, B.mean(loss))
        return [d, s]
    sched = schedule(running)
    assert not any(w.startswith("p") for w in sched[0]["writes"])


def test_losses_of_many_workgroups_are_summed_by_a_launch_of_their_own():
    """128 workgroups of 16 rows, and one more."""
    assert kinds(schedule(lambda B, mk: losses(B, mk, rows=2048))) == ["ROWOP"]
    assert kinds(schedule(lambda B, mk: losses(B, mk, rows=2049))) == ["ROWOP", "ALL"]


# ---- scalings round an attention core --------------------------------------------------------------------
def core(B, mk, form=""):
    b, s, h, d = 2, 40, 2, 64
    split = lambda t: B.permute(B.reshape(t, (b, s, h, d)), (0, 2, 1, 3))                     # noqa: E731
    merge = lambda t: B.reshape(B.permute(t, (0, 2, 1, 3)), (b * s, h * d))                   # noqa: E731
    q, k, v, dy = (mk((b * s, h * d), "bf16", form == "overwritten" and i == 0) for i in range(4))
    qs = B.mul(q, 0.125)
    qh, kh, vh, dh = (split(t) for t in (qs, k, v, dy))
    p = B.softmax(B.matmul(qh, kh, trans_b=True))
    ds = B.softmax_grad(B.matmul(dh, vh, trans_b=True), p)
    dq = merge(B.matmul(ds, kh))
    out = [merge(B.matmul(p, vh)), B.mul(dq, 0.125), merge(B.matmul(ds, qh, trans_a=True)), merge(B.matmul(p, dh, trans_a=True))]
    if form == "queries held":
        out.append(qs)
    elif form == "view held":
        out.append(B.reshape(qs, (b * s * h, d)))
    elif form == "gradient held":
        out.append(dq)
    elif form == "another core":
        p2 = B.softmax(B.matmul(qh, vh, trans_b=True))
        out.append(merge(B.matmul(p2, kh)))
    elif form == "keys too":
        p2 = B.softmax(B.matmul(kh, qh, trans_b=True))
        out.append(merge(B.matmul(p2, vh)))
    elif form == "overwritten":
        B.assign(q, B.add(q, 1.0))
        out.append(q)
    return out


def test_a_cores_scalings_ride():
    sched = schedule(core)
    assert kinds(sched) == ["ATTN"] * 3
    assert all(sum(r.startswith("p") for r in l["reads"]) == n for l, n in zip(sched, (3, 4, 4)))     # (the queries as they were)


@pytest.mark.parametrize("form", ["queries held", "view held", "another core", "keys too", "overwritten"])
def test_scaled_queries_that_others_see_are_in_memory(form):
    """The host holds them or a view of them, another core reads them, as queries or as keys; the unscaled ones change in the same step."""
    sched = schedule(lambda B, mk: core(B, mk, form))
    cores = [l for l in sched if l["kind"] == "ATTN"]
    scaling = sched[0]
    assert scaling["kind"] == "EW" and len(cores) == (4 if form in ("another core", "keys too") else 3)
    assert all(scaling["writes"] <= l["reads"] and not scaling["reads"] & l["reads"] for l in cores)
    assert sum(l["kind"] == "EW" for l in sched) == (2 if form == "overwritten" else 1)


def test_a_query_gradient_that_the_host_holds_is_in_memory():
    sched = schedule(lambda B, mk: core(B, mk, "gradient held"))
    assert kinds(sched).count("EW") == 1 and kinds(sched)[:2] == ["ATTN"] * 2
    (scaling,) = [l for l in sched if l["kind"] == "EW"]
    assert any(scaling["reads"] <= l["writes"] for l in sched if l["kind"] == "ATTN")
