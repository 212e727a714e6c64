"""Fused calls of at most 8 ranks in registers: every p and tree layout, every
operator, sizes around a wavefront's 128 quanta, trailing elements (in the last
run of quanta or in a launch of their own), unaligned rows, in place; bit for
bit against the oracle, and the rows between which it is not used."""

import numpy as np
import pytest
import torch

from oracle import c_oracle
from tests._gpu import _Env, assert_all_ranks_equal, env_unit, lib, need_gpu

pytestmark = pytest.mark.gpu


def _data(dtype, p, m):
    r = np.random.default_rng(4300 + p)
    if dtype == "float32":
        return r.standard_normal((p, m), np.float32)
    if dtype == "int32":
        return r.integers(-1 << 31, 1 << 31, (p, m), dtype=np.int32)
    return r.integers(0, 1 << 32, (p, m, 4), dtype=np.uint32)


@pytest.mark.parametrize("dtype,op", [("int32", "sum"), ("int32", "max"),
                                      ("float32", "sum"),
                                      ("u32mat2x2", "matmul")])
@pytest.mark.parametrize("alg", ["dual", "single", "reduce_bcast"])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6, 7, 8])
def test_every_tree(p, alg, dtype, op, capfd):
    need_gpu()
    dpar = lib()
    words = 4 if dtype == "u32mat2x2" else 1
    s = torch.cuda.current_stream()
    # quanta: 1, 127, 128, 129, 512, 513; then 4 m' + 1 .. 3 elements (more than
    # 24 MB moved, below which such calls take one element per lane): whole
    # quanta that fill their last run of 128, so that the trailing elements
    # are a launch of their own, and that leave 1, 64 or 127 in it, so that
    # they ride there as a quantum that overlaps the one before
    sizes = [4, 508, 512, 516, 2048, 2052]
    if words == 1 and p == 8 and alg != "reduce_bcast":
        full = [400385, 399874, 399875, 399361]
        rides = [4 * 100097 + 1, 4 * 100160 + 2, 4 * 100095 + 3]
        assert [m // 4 % 128 for m in full] == [0] * 4
        assert [m // 4 % 128 for m in rides] == [1, 64, 127]
        sizes += full + rides
    for m in sizes:
        x = _data(dtype, p, m)
        want = c_oracle.allreduce(x, dtype, op,
                                  layout="dual" if alg == "dual" else "single",
                                  threads=8)
        flat = np.ascontiguousarray(x).view(np.int32).reshape(p, -1)
        n = flat.shape[1]
        for offset, in_place in ((0, False), (1, False), (3, True)):
            big = torch.full((p, n + 8), -7, dtype=torch.int32, device="cuda")
            big[:, offset:offset + n] = torch.from_numpy(flat).cuda()
            out = big if in_place else torch.full_like(big, -7)
            with env_unit(None), _Env("DPAR_LOG", 1):
                dpar.dpar_allreduce_opt(
                    dpar.rows(big[:, offset:]), dpar.rows(out[:, offset:]), p,
                    m, dtype, op, 1, alg, "auto", 0, -1, s)
            dpar.dpar_check_status(s)
            err = capfd.readouterr().err
            assert "in_registers" in err, err
            got = out.cpu().numpy()
            assert (got[:, :offset] == -7).all()
            assert (got[:, offset + n:] == -7).all()
            got = np.ascontiguousarray(got[:, offset:offset + n])
            assert_all_ranks_equal(got.view(x.dtype).reshape(x.shape), want,
                                   f"p={p} m={m} {alg} +{offset}")


@pytest.mark.parametrize("p,m,few", [
    (8, 1 << 20, True),            # one wide item per CU
    (8, (1 << 20) + 4, False),
    (3, (1 << 23) - 4, False),     # rows below 32 MB
    (3, 1 << 23, True),
    (3, (1 << 23) + 1, True),      # a full run, then one trailing element
    (9, 1 << 18, False),
])
def test_rule_edges(p, m, few, capfd):
    need_gpu()
    dpar = lib()
    x = torch.randint(-1000, 1000, (p, m), dtype=torch.int32, device="cuda")
    y = torch.zeros_like(x)
    s = torch.cuda.current_stream()
    with env_unit(None), _Env("DPAR_LOG", 1):
        dpar.dpar_allreduce(dpar.rows(x), dpar.rows(y), p, m, "int32", "sum",
                            0, s)
    dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    assert ("in_registers" in err) == few, err
    assert bool((y == x.sum(0, dtype=torch.int64).to(torch.int32)).all())


# a little more than one of its workgroups per CU: post-order items in full
# chunks from 5 ranks on (8 in place), 8 to 13 of them per CU, without trailing
# elements; long rows off the 128-byte lines: wide items with 3 to 6 ranks
@pytest.mark.parametrize("p,m,off,kernel", [
    (4, (1 << 19) + 4, 0, "few_ranks"),
    (5, 1 << 19, 0, "few_ranks"),
    (5, (1 << 19) + 4, 0, "postorder"),
    (5, 9 << 16, 0, "postorder"),
    (5, 608 << 10, 0, "few_ranks"),        # three chunks a block
    (8, 12 << 16, 3, "postorder"),
    (8, 800 << 10, 0, "few_ranks"),
    (8, (12 << 16) - 1, 0, "few_ranks"),
    (7, 9 << 16, None, "few_ranks"),       # in place
    (8, 9 << 16, None, "postorder"),
    (2, 1 << 23, 1, "few_ranks"),
    (3, 1 << 23, 0, "few_ranks"),
    (3, 1 << 23, 4, "wide"),
    (6, 1 << 23, 1, "wide"),
    (4, (1 << 23) + 2, 1, "few_ranks"),
    (6, (1 << 23) + 2, 1, "wide"),
    (7, 1 << 23, 1, "few_ranks"),
])
def test_rule_exceptions(p, m, off, kernel, capfd):
    need_gpu()
    dpar = lib()
    in_place, off = off is None, off or 0
    ld = -(-m // 32) * 32 + 32
    x = torch.randint(-1000, 1000, (p, ld), dtype=torch.int32, device="cuda")
    x[:, :off] = 0
    x[:, off + m:] = 0
    want = x[:, off:off + m].sum(0, dtype=torch.int64).to(torch.int32)
    y = x if in_place else torch.zeros_like(x)
    s = torch.cuda.current_stream()
    with env_unit(None), _Env("DPAR_LOG", 1):
        dpar.dpar_allreduce(dpar.rows(x[:, off:]), dpar.rows(y[:, off:]), p,
                            m, "int32", "sum", 0, s)
    dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    assert f" kernel={kernel}\n" in err, err
    assert bool((y[:, off:off + m] == want).all())
    assert bool((y[:, :off] == 0).all() and (y[:, off + m:] == 0).all())
