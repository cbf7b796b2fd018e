"""What the host side launches, and on which streams and scratch, recorded
without a GPU (hip_recorder.py)."""
import pytest

import hip_recorder


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return hip_recorder.build(str(tmp_path_factory.mktemp("hip_recorder")))


@pytest.mark.parametrize("many", [False, True])
def test_adjoint_takes_the_tangents_threads_per_cell(lib, many):
    """Every size bucket, with the default variants and with each variant that
    a caller may set for it."""
    out = hip_recorder.run(lib, """
MANY = %d
h, res = ctx(), []
cap = [128, 256, 512, 1024, 2048, 4096, 32768]
for b in range(7):
    p = Pop([min(cap[b], 5000)] + [1] * (300 if MANY else 0))
    for v in range(-1, 16):
        if L.mcc_set_variant(h, b, v) != 0:
            continue
        log()
        assert jvp(h, p) == 0 and adjoint(h, p) == 0
        x = log()
        # the bucket's own launch: in the tangent form, largest first, after those of the
        # larger buckets that n particles could reach; the adjoint's largest is its last
        above = sum(p.n > cap[k - 1] for k in range(b + 1, 7))
        tan, adj = steps(x)[above], steps(x, "adjoint_kernel")[-1]
        res.append((b, v, tan["block"], adj["block"]))
        L.mcc_set_variant(h, b, -1)
print(json.dumps(res))
""" % many)
    assert len(out) > 40
    assert [x for x in out if x[2] != x[3]] == []


def _joined(lines):
    """Every stream that was forked from the caller's (0) and launched on is
    joined to it afterwards: an event recorded on it after its last launch and
    waited for by stream 0."""
    for s in {x["stream"] for x in lines if x["op"] == "wait" and x["stream"] != 0}:
        last = max((i for i, x in enumerate(lines) if x["op"] in ("launch", "wait")
                    and x["stream"] == s))
        rec = [i for i, x in enumerate(lines) if i > last and x["op"] == "record"
               and x["stream"] == s]
        if not rec or not any(x["op"] == "wait" and x["stream"] == 0
                              and x["event"] == lines[rec[0]]["event"] for x in lines[rec[0]:]):
            return False
    return True


def test_streams_are_joined_after_an_error(lib):
    """A launch that fails behind the fork, and a scratch allocation that
    fails: the call reports it, no kernel stays unordered with the caller's
    stream, and a failed allocation leaves nothing launched."""
    out = hip_recorder.run(lib, """
h, res = ctx(), []
p = Pop([2000] * 10 + [300] * 10 + [50] * 300)
for k in range(1, 10):
    sorted_step(h, p); log()
    rt.rec_fail_launch(k)
    res.append((sorted_step(h, p), log()))
    rt.rec_fail_launch(0)
rt.hipGetLastError()
h = ctx()
L.mcc_set_variant(h, 0, 10)        # (700 MB of scratch)
rt.rec_malloc_limit(1 << 20); log()
rc = sorted_step(h, p)
print(json.dumps([res, rc, log()]))
""")
    res, rc, lines = out
    assert [r for r, _ in res] == [-3] * 9  # (two front kernels, seven buckets)
    for r, x in res:
        assert _joined(x), (r, x)
    assert sum(1 for r, x in res if r == -3 and any(y["op"] == "launch" and y["stream"] != 0
                                                    for y in x)) >= 2
    assert rc == -2 and not any("collide_kernel" in y.get("kernel", "") for y in lines)
    assert _joined(lines)


@pytest.mark.parametrize("cell,used_before", [(100, 478e6), (1000, 478e6), (1500, 478e6),
                                              (4000, 478e6), (8000, 1912e6)])
def test_adjoint_fits_where_it_fitted(lib, cell, used_before):
    """Seven collisions with no more memory than 228 B per particle of the 4096
    (two workgroups per compute unit) or 32768 kernels' capacity: accepted, in
    smaller groups of records; refused with less than one record's."""
    out = hip_recorder.run(lib, """
cell, used = %d, %d
h, p = ctx(), Pop([cell] * 600, collisions=((0, 0),) * 7)
rt.rec_malloc_limit(used); log()
rc = adjoint(h, p)
big = [x["bytes"] for x in log() if x["op"] == "malloc" and x["ok"] and x["bytes"] > 1e6]
h2 = ctx()
rt.rec_malloc_limit(100000)
print(json.dumps([rc, big, adjoint(h2, p)]))
""" % (cell, used_before))
    assert out[0] == 0 and out[1] and max(out[1]) <= used_before
    assert out[2] == -2


def test_streams_are_created_when_first_needed(lib):
    """A context creates one side stream, calls none, a plan its capture's, and
    the context's second side stream at the first plan that takes three."""
    out = hip_recorder.run(lib, """
def made():
    x = log()
    return [sum(y["op"] == o for y in x) for o in ("stream", "event")]

h, res = ctx(), []
res.append(made())
sorted_step(h, Pop([50] * 20)); res.append(made())
a = plan(h, Pop([50] * 20)); res.append(made())
b = plan(h, Pop([50] * 400 + [200] * 20)); res.append(made())
sorted_step(h, Pop([50] * 400)); res.append(made())
sorted_step(h, Pop([50] * 400)); res.append(made())
c = plan(h, Pop([50] * 400 + [200] * 20 + [400])); res.append(made())
h = ctx(); made()
d = plan(h, Pop([50, 200, 400, 1000] * 99)); res.append(made())
print(json.dumps([res, [x[0] for x in (a, b, c, d)]]))
""")
    assert out[0] == [[1, 2], [0, 0], [1, 0], [1, 0], [0, 0], [0, 0], [2, 1], [2, 1]]
    assert out[1] == [0] * 4


@pytest.mark.parametrize("sizes,streams", [
    ([1500] * 20 + [3000] * 20, 2), ([1500] * 20 + [900] * 20, 1), ([3000] * 20 + [900] * 20, 1),
    ([1500] * 20, 1), ([1500] * 20 + [3000] * 20 + [900], 3), ([100] * 400 + [200] * 400, 1),
    ([1500] * 800 + [3000] * 400 + [900], 2)])
def test_streams_of_a_plan(lib, sizes, streams):
    """The streams that a plan's kernels are dealt to: two for cells of
    1025-2048 and 2049-4096 alone, one for another pair, else by the number of
    buckets and particles; all joined."""
    lines = hip_recorder.run(lib, """
h, p = ctx(), Pop(%r)
log()
rc, q = plan(h, p)
assert rc == 0
print(json.dumps(log()))
""" % sizes)
    start = [i for i, x in enumerate(lines) if x["op"] == "stream"][-1]  # (the capture's)
    cs = lines[start]["id"]
    used = {x["stream"] for x in lines[start:] if "collide_kernel" in x.get("kernel", "")}
    assert len(used) == streams and (streams == 1 or cs in used)
    for x in lines:
        x["stream"] = 0 if x.get("stream") == cs else x.get("stream", -1)
    assert _joined(lines[start:])


@pytest.mark.parametrize("n,n_cells,passes,records", [
    (5000, 511, 1, False), (5000, 512, 2, False), (5000, (1 << 18) - 1, 2, False),
    (5000, 1 << 18, 3, True), ((1 << 24) - 1, 1 << 18, 3, True), (1 << 24, 1 << 18, 3, False),
    (5000, (1 << 27) - 1, 3, True), (5000, 1 << 27, 4, True)])
def test_route_of_the_unsorted_payload(lib, n, n_cells, passes, records):
    """With the keys through one and two radix passes, as records from three up
    below 2^24 particles, and with four."""
    lines = hip_recorder.run(lib, """
h = ctx()
log()
assert collide(h, %d, %d) == 0
print(json.dumps(log()))
""" % (n, n_cells))
    count = lambda k: sum(k in x.get("kernel", "") for x in lines)
    assert count("k_radix_hist") == passes
    assert count("k_radix_move") == count("k_move_back") == (0 if records else passes)
    assert count("k_radix_scatter") == (passes if records else 0)
    assert count("k_gather_rec") == count("k_scatter_rec") == (1 if records else 0)


@pytest.mark.parametrize("size,cells,aside", [
    (700, 2048, False), (700, 2049, True), (512, 2049, False), (513, 2049, True),
    (1024, 2049, True), (1025, 2049, False), (100, 40960, False), (100, 40961, True),
    (128, 40961, True), (129, 40961, False), (300, 3000, False)])
def test_side_stream_of_a_call(lib, size, cells, aside):
    """The buckets that a call puts on its side stream: every other one, or the
    2048 and 4096 buckets alone for many cells whose mean is in the 1024 bucket
    or, for very many, in the 128 bucket."""
    caps = [128, 256, 512, 1024, 2048, 4096, 32768]
    lines = hip_recorder.run(lib, """
h, p = ctx(), Pop([%d] * %d)
log()
assert sorted_step(h, p) == 0
print(json.dumps(steps(log())))
""" % (size, cells))
    cap = [int(x["kernel"].split("ELi")[1].split("E")[0]) for x in lines]
    assert cap == sorted(caps, reverse=True)
    side = {c for c, x in zip(cap, lines) if x["stream"] != 0}
    assert side == ({2048, 4096} if aside else {4096, 1024, 256})


@pytest.mark.parametrize("sizes,form,block", [
    ([64] * 20, {}, 64), ([65] * 20, {}, 256), ([60] * 20 + [100], {}, 256),
    ([60] * 20 + [300], {}, 64), ([60] * 257, {}, 64), ([100] * 257, {}, 64),
    ([64], dict(precision=1), 64), ([60] * 20, dict(precision=1, pairing=1), 256),
    ([60] * 20, dict(pairing=1), 64)])
def test_threads_of_a_plan_of_few_small_cells(lib, sizes, form, block):
    lines = hip_recorder.run(lib, """
h, p = ctx(), Pop(%r)
log()
rc, q = plan(h, p, native.make_params(**%r))
assert rc == 0
print(json.dumps(steps(log())))
""" % (sizes, form))
    assert lines[-1]["block"] == block  # (the smallest bucket, launched last)
