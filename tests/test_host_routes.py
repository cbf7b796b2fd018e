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
