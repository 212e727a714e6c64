"""Level work items (groups of at most 7 ranks per thread) at the sizes where
a cut, a remainder or a rule can go wrong: bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import synth
from oracle import c_oracle
from tests._gpu import _Env, assert_all_ranks_equal, env_unit, lib, need_gpu

pytestmark = pytest.mark.gpu


def _run(x, dtype, op, b=0, alg="dual", exec="auto", in_place=False,
         offset=0):
    """Rows `offset` words past the start of a row of a padded buffer; the
    words around every output row must stay as they were."""
    dpar = lib()
    p = x.shape[0]
    flat = np.ascontiguousarray(x).view(np.int32).reshape(p, -1)
    n = flat.shape[1]
    big = torch.full((p, n + 8), -7, dtype=torch.int32, device="cuda")
    big[:, offset:offset + n] = torch.from_numpy(flat).cuda()
    out = big if in_place else torch.full_like(big, -7)
    s = torch.cuda.current_stream()
    xs = dpar.rows(big[:, offset:])
    ys = dpar.rows(out[:, offset:])
    dpar.dpar_allreduce_opt(xs, ys, p, x.shape[1], dtype, op, b, alg, exec,
                            0, -1, s)
    dpar.dpar_check_status(s)
    assert bool((out[:, :offset] == -7).all().item())
    assert bool((out[:, offset + n:] == -7).all().item())
    got = out[:, offset:offset + n].cpu().numpy()
    return np.ascontiguousarray(got).view(x.dtype).reshape(x.shape)


def _want(x, dtype, op, alg="dual"):
    return c_oracle.allreduce(x, dtype, op, layout=alg, threads=8)


# chunk lengths 4 .. 64 quanta, a last chunk of one quantum, of all but one,
# and full; trailing elements next to each; groups that fill, overfill and
# leave idle the threads
@pytest.mark.parametrize("m", [1 << 14, (1 << 14) + 4, (1 << 14) - 4,
                               (1 << 14) + 1, (1 << 14) + 7, 65539])
@pytest.mark.parametrize("p", [17, 100, 255, 257])
@pytest.mark.parametrize("alg", ["dual", "single"])
def test_one_launch_cuts(p, m, alg):
    need_gpu()
    x = np.random.default_rng(4000 + p).standard_normal((p, m), np.float32)
    want = _want(x, "float32", "sum", alg)
    for exec in ("auto", "split"):
        for offset, in_place in ((0, False), (1, True)):
            got = _run(x, "float32", "sum", 0, alg, exec, in_place, offset)
            assert_all_ranks_equal(got, want, f"{alg} {exec} p={p} m={m} "
                                   f"+{offset} in_place={in_place}")


@pytest.mark.parametrize("dtype,op,dist", [
    ("int32", "sum", "uniform_int"), ("int32", "max", "uniform_int"),
    ("float32", "sum", "normal_f32"), ("u32mat2x2", "matmul",
                                       "odd_det_u32_mat")])
@pytest.mark.parametrize("p,m", [(3, 64), (7, 1000), (8, 1001), (15, 64),
                                 (36, 8374), (64, 4096), (1153, 258),
                                 (4099, 65)])
@pytest.mark.parametrize("exec", ["auto", "split", "ticket", "launch",
                                  "rounds"])
def test_types_in_place(p, m, dtype, op, dist, exec):
    """The library's chunk and 64 quanta (a wavefront per group)."""
    need_gpu()
    kw = {"lo": -1000, "hi": 1000} if dist == "uniform_int" else {}
    x = synth.generate(dist, 4100 + p, p, m, **kw)
    for alg in ("dual", "single"):
        want = _want(x, dtype, op, alg)
        for lg in (None, 6):
            with env_unit("level"), _Env("DPAR_LEVEL_LOG2T", lg):
                got = _run(x, dtype, op, 3, alg, exec,
                           in_place=exec != "rounds")
            assert_all_ranks_equal(got, want, f"{dtype} {alg} {exec} p={p}")


# edges of the rules: level items up to one 1 KB chunk per CU below 256
# ranks, subtree items up to two per CU, fused up to 256 MB moved and with
# pieces of 512 bytes on rows off the 128-byte lines
@pytest.mark.parametrize("p,m,pad,want", [
    (200, 65536, 0, "exec=one_launch_fused unit=level"),
    (200, 65540, 0, "unit=postorder"),
    (16, 65536, 0, "unit=postorder"),
    (300, 111852, 0, "exec=split unit=subtree"),
    (300, 111848, 0, "exec=one_launch_fused unit=subtree"),
    (1152, 16384, 1, "exec=split unit=subtree"),
    (600, 20000, 1, "exec=one_launch_fused unit=subtree"),
    (300, 131072, 0, "exec=split unit=subtree"),
    (300, 131076, 0, "unit=postorder"),
])
def test_rule_edges(p, m, pad, want, capfd):
    need_gpu()
    dpar = lib()
    x = torch.randint(-1000, 1000, (p, m + pad), dtype=torch.int32,
                      device="cuda")
    y = torch.zeros_like(x)
    s = torch.cuda.current_stream()
    with env_unit(None), _Env("DPAR_LOG", 1):
        dpar.dpar_allreduce(dpar.rows(x), dpar.rows(y), p, m, "int32", "sum",
                            0, s)
        dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    assert want in err, err[-400:]
    assert ("level_chunk_quanta" in err) == ("postorder" not in want)
    total = x[:, :m].sum(0, dtype=torch.int64).to(torch.int32)
    assert bool((y[:, :m] == total).all().item())
    assert bool((y[:, m:] == 0).all().item())
