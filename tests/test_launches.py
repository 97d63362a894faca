"""What the launches of a plan read and write (lt_dump_schedule), against its regions (lt_dump_plan): regions are
regrouped, dropped and merged on their way to launches (the attention core, reshaped results, sums that ride
along, updates and finalisers in a second launch), and none of it may change what a launch finds in memory."""
import numpy as np
import pytest

from paper_2102_13267_amd import Context
from plan_check import DEVICE_DATA, EXPAND, NARROW, PERMUTE, RESHAPE, parse_key, parse_plan
from test_plan_validity import c1, c2, c3, c4, c5, random_trace
from test_schedule import parse


class LaunchError(AssertionError):
    pass


def check_launches(key, n_nodes, plan, sched):
    """1. a temporary is written by a launch before the first launch that reads it;
    2. a parameter is written only if the plan updates it in place, and every such update has a launch;
    3. no launch of a region that reads a parameter's old value comes behind one of another region that overwrites it."""
    regions, (nodes, _) = parse_plan(plan), parse_key(key, n_nodes)

    def need(cond, msg):
        if not cond:
            raise LaunchError(msg)
    computed = {m for r in regions for m in r["members"]}

    def base(v):                                     # through views
        while v[0] not in computed and nodes[v[0]].op in (EXPAND, RESHAPE, PERMUTE, NARROW):
            v = nodes[v[0]].ins[0]
        return v
    old = [{f"p{nodes[base(v)[0]].ordinal}" for v in r["inputs"] if nodes[base(v)[0]].op == DEVICE_DATA} for r in regions]
    updates = {f"p{p}" for r in regions for (_, p) in r["inplace"]}
    written = {}
    for l in sched:
        # (the launches of an attention core stand for several regions)
        stale = set().union(*old) if l["kind"] == "ATTN" else old[l["region"]]
        for s in l["reads"]:
            if s[0] == "t":
                need(s in written, f"L{l['i']} reads {s} before anything has written it")
            else:
                need(s not in stale or written.get(s, l["region"]) == l["region"], f"L{l['i']} of R{l['region']} reads {s} after R{written.get(s)} has overwritten it")
        for s in l["writes"]:
            need(s[0] == "t" or s in updates, f"L{l['i']} writes {s}, which the plan does not update in place")
            written.setdefault(s, l["region"])
    need(updates <= set(written), "an update in place has no launch")


def launches(build):
    ctx = Context()
    keep = build(ctx, lambda shape, dtype="f32", donatable=False: ctx.tensor(
        np.zeros(shape, {"s32": np.int32}.get(dtype, np.float32)), dtype=dtype, donatable=donatable))
    info = ctx.barrier()
    out = ctx.dump_key(), info.n_nodes, ctx.dump_plan(), parse(ctx.dump_schedule())
    del keep
    return out


def attention(B, mk, update=False):
    """The core, with q, k and v updated in place by what their own gradients give when `update`."""
    split = lambda t: B.permute(B.reshape(t, (2, 40, 2, 64)), (0, 2, 1, 3))                    # noqa: E731
    merge = lambda t: B.reshape(B.permute(t, (0, 2, 1, 3)), (80, 128))                        # noqa: E731
    q, k, v, dy = (mk((80, 128), "bf16", True) for _ in range(4))
    qh, kh, vh, dh = (split(t) for t in (q, k, v, dy))
    p = B.softmax(B.matmul(qh, kh, trans_b=True))
    out = [merge(B.matmul(p, vh))]
    ds = B.softmax_grad(B.matmul(dh, vh, trans_b=True), p)
    for t, g in ((q, merge(B.matmul(ds, kh))), (k, merge(B.matmul(ds, qh, trans_a=True))), (v, merge(B.matmul(p, dh, trans_a=True)))):
        if update:
            B.assign(t, B.sub(t, B.mul(g, 0.1)))
        out.append(g)
    if update:
        B.assign(dy, B.mul(dy, 0.5))
    return out + [q, k, v, dy]


def norm(B, mk):
    """Weight and bias gradient of a norm, both parameters updated in place."""
    x, dy, w, b = mk((64, 128)), mk((64, 128)), mk((128,), "f32", True), mk((128,), "f32", True)
    y, mu, rs = B.layer_norm(x, w, b, eps=1e-5)
    xhat = B.mul(B.sub(x, B.reshape(mu, (64, 1))), B.reshape(rs, (64, 1)))
    B.assign(w, B.sub(w, B.sum(B.mul(dy, xhat), axis=0)))
    B.assign(b, B.sub(b, B.sum(dy, axis=0)))
    return [y, w, b]


def second_launches(B, mk):
    """A finaliser and an optimiser update in launches of their own, and a reshaped result."""
    x, w, m, v = mk((200, 300), "bf16"), mk((300, 260), "bf16", True), mk((300, 260), "f32", True), mk((300, 260), "f32", True)
    g = B.matmul(x, mk((200, 260), "bf16"), trans_a=True)
    m1, v1 = B.add(B.mul(m, 0.9), g, alpha=0.1), B.add(B.mul(v, 0.99), B.square(g), alpha=0.01)
    B.assign(w, B.cast(B.sub(w, B.div(m1, B.add(B.sqrt(v1), 1e-8))), "bf16"))
    B.assign(m, m1)
    B.assign(v, v1)
    t, s = mk((4096,)), mk((), "f32", True)
    r = B.add(B.mul(s, 0.9), B.amax(B.abs(t)))
    B.assign(s, r)
    return [w, m, v, s, B.div(t, r), B.reshape(B.softmax(B.matmul(x, w)), (260, 200))]


@pytest.mark.parametrize("build", [c1, c2, c3, c4, c5, attention, lambda B, mk: attention(B, mk, True), norm, second_launches])
def test_launches_of_programs(build):
    check_launches(*launches(build))


def test_random_traces():
    for seed in range(400):
        try:
            args = launches(random_trace(seed))
        except Exception as e:
            if type(e).__name__ == "LtError" and e.status == 5 and "internal" not in str(e):
                continue
            raise
        check_launches(*args)


def test_planted_mistakes_are_seen():
    key, n, plan, sched = launches(lambda B, mk: attention(B, mk, True))
    kinds = [l["kind"] for l in sched]
    assert kinds.count("ATTN") == 3
    assert [l["writes"] & {"p0", "p1", "p2", "p3"} == set() for l in sched[:3]] == [True] * 3
    for bad in ([sched[i] for i in (2, 0, 1)] + sched[3:],                             # dk and dv before what they are rebuilt from
                sched[:2] + sched[3:] + sched[2:3],                                   # updates of q, k, v before dk and dv
                sched[:-1],                                                           # an update that never runs
                [dict(l, writes=l["writes"] | {"p3"}) if l["kind"] == "ATTN" else l for l in sched[:1]] + sched[1:]):
        with pytest.raises(LaunchError):
            check_launches(key, n, plan, [dict(l, i=i) for i, l in enumerate(bad)])
