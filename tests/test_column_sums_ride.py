"""Column sums that ride with the contraction of the same tensor (host logic, null device): which do, which must not."""
import pytest

from test_merged_launches import kinds, schedule


def gradients(reduce="sum", dt="bf16", rows=512, cols=(1024, 1024), sum_first=False, between=None, update=False, other=False):
    """dW = x^T dy and the column sums of dy."""
    def build(B, mk):
        x, dy, z = mk((rows, cols[0]), dt), mk((rows, cols[1]), dt, True), mk((rows, cols[1]), dt)
        b = mk((cols[1],), dt, True)
        total = lambda: getattr(B, reduce)(z if other else dy, axis=0)          # noqa: E731
        db = total() if sum_first else None
        dw = B.matmul(x, dy, trans_a=True)
        out = [dw] if not sum_first else [db, dw]
        if between:
            out += between(B, dy, b)
        if not sum_first:
            db = total()
            out.append(db)
        if update:
            B.assign(b, B.sub(b, db))
        return out + [x, dy, z, b]
    return build


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("reduce", ["sum", "mean"])
@pytest.mark.parametrize("sum_first", [False, True])
@pytest.mark.parametrize("update", [False, True])
def test_they_ride(dt, reduce, sum_first, update):
    """One launch in an unsplit product (its workgroups' halves share k)."""
    sched = schedule(gradients(reduce, dt, rows=1024, cols=(2048, 2048) if dt == "bf16" else (1024, 2048), sum_first=sum_first, update=update))
    assert kinds(sched) == ["MM"]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_partial_sums_of_a_split_product_are_added_up(dt):
    sched = schedule(gradients(dt=dt, rows=8192, cols=(1024, 512)))
    assert sorted(kinds(sched)) == ["COL", "MM", "SPLITPOST"]
    (col,) = [l for l in sched if l["kind"] == "COL"]
    (mm,) = [l for l in sched if l["kind"] == "MM"]
    assert len(col["reads"]) == 1 and set(col["reads"]) <= set(mm["writes"])


@pytest.mark.parametrize("case", [dict(reduce="amax"), dict(other=True), dict(cols=(1024, 64)),
                                  dict(rows=8192, cols=(512, 514), dt="f32")])     # (split, no whole chunks)
def test_they_keep_their_launch(case):
    sched = schedule(gradients(**case))
    (col,) = [l for l in sched if l["kind"] == "COL"]
    assert not any(set(col["reads"]) & set(l["writes"]) for l in sched)


def test_sums_of_an_overwritten_tensor_keep_their_launch():
    def update(B, dy, b):
        B.assign(dy, B.mul(dy, 0.5))
        return [dy]
    sched = schedule(gradients(between=update))
    assert "COL" in kinds(sched)


def test_sums_whose_parameter_is_read_in_between_are_not_early():
    """What replaces b is launched behind the product that still reads it."""
    def read(B, dy, b):
        return [B.matmul(B.reshape(b, (1, 1024)), dy, trans_b=True)]
    sched = schedule(gradients(cols=(1024, 1024), rows=1024, between=read, update=True))
    writer = [i for i, l in enumerate(sched) if "p3" in l["writes"] or any(w.startswith("p") for w in l["writes"])]
    readers = [i for i, l in enumerate(sched) if set(sched[writer[-1]]["writes"]) & set(l["reads"])]
    assert max(readers) <= writer[-1]


@pytest.mark.parametrize("rows,cols,rides", [(16384, (4096, 4096), True), (16392, (4096, 4096), False), (65536, (1024, 8192), False),
                                             (65536, (2048, 2048), True), (16392, (4100, 4100), True)])
def test_longest_bf16_products(rows, cols, rides):
    """Beyond 2^38 multiply-adds an unsplit product in whole tiles, whose workgroups are no halves, is slower with the sums than without."""
    assert kinds(schedule(gradients(rows=rows, cols=cols))) == ["MM"] + ([] if rides else ["COL"])
