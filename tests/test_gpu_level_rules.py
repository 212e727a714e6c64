"""Rules of the level work item, each at the sizes where it turns, shown by the
plan line; bit for bit against the oracle."""

import numpy as np
import pytest
import torch

from oracle import c_oracle
from tests._gpu import _Env, assert_all_ranks_equal, env_unit, lib, need_gpu

pytestmark = pytest.mark.gpu


def _call(p, m, dtype, exec, b, pad, capfd):
    dpar = lib()
    words = 4 if dtype == "u32mat2x2" else 1
    op = "matmul" if words == 4 else "sum"
    r = np.random.default_rng(6100 + p)
    if dtype == "float32":
        x = r.standard_normal((p, m), np.float32)
    elif words == 4:
        x = r.integers(0, 1 << 32, (p, m, 4), dtype=np.uint32)
    else:
        x = r.integers(-1 << 31, 1 << 31, (p, m), dtype=np.int32)
    flat = np.ascontiguousarray(x).view(np.int32).reshape(p, -1)
    n = flat.shape[1]
    big = torch.full((p, n + pad), -7, dtype=torch.int32, device="cuda")
    big[:, :n] = torch.from_numpy(flat).cuda()
    out = torch.full_like(big, -7)
    s = torch.cuda.current_stream()
    with env_unit(None), _Env("DPAR_LOG", 1):
        dpar.dpar_allreduce_ex(dpar.rows(big), dpar.rows(out), p, m, dtype,
                               op, b, exec, s)
    dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    got = out.cpu().numpy()
    assert (got[:, n:] == -7).all()
    got = np.ascontiguousarray(got[:, :n]).view(x.dtype).reshape(x.shape)
    want = c_oracle.allreduce(x, dtype, op, layout="dual", threads=8)
    assert_all_ranks_equal(got, want, f"{p} {m} {dtype} {exec}")
    return err


# 4-byte lanes: one turn of 512 places, at most 8 quanta; then longer chunks
# from 160 items on; 16-byte lanes: one turn of 1024 places, 4 quanta with more
# items than an eighth of the CUs, whole lines from half an item per CU on
@pytest.mark.parametrize("p,m,dtype,exec,quanta", [
    (64, 33, "float32", "auto", 8),
    (288, 1, "float32", "auto", 8),
    (1152, 33, "int32", "auto", 2),
    (4608, 7, "float32", "auto", 1),
    (4608, 255, "float32", "auto", 1),
    (4608, 257, "float32", "auto", 2),
    (6000, 5, "float32", "split", 1),
    (4608, 3, "u32mat2x2", "auto", 1),
    (4608, 33, "u32mat2x2", "auto", 2),
    (4608, 65, "u32mat2x2", "auto", 4),
    (2304, 512, "u32mat2x2", "auto", 8),
    (2304, 508, "u32mat2x2", "auto", 4),
    (6000, 128, "u32mat2x2", "auto", 8),
    (6000, 124, "u32mat2x2", "auto", 4),
    (288, 2001, "float32", "auto", 16),
    (1152, 1301, "float32", "launch", 16),
    (1152, 2049, "float32", "auto", 16),
    (1152, 2045, "float32", "auto", 8),
    (1152, 5615, "float32", "rounds", 16),
    (288, 5615, "float32", "rounds", 32),
    (1152, 1024, "u32mat2x2", "auto", 4),
    (4608, 27, "u32mat2x2", "launch", 1),
    (2304, 217, "float32", "rounds", 1),
    (2304, 257, "float32", "rounds", 2),
    (2304, 13, "int32", "ticket", 8),
    (320, 1563, "float32", "ticket", 16),
])
def test_chunk(p, m, dtype, exec, quanta, capfd):
    need_gpu()
    err = _call(p, m, dtype, exec, 1, 0, capfd)
    assert f" level_chunk_quanta={quanta} " in err, err


# the cooperative executors: few workgroups at the barrier, few turns each
@pytest.mark.parametrize("exec,p,m,b,quanta", [
    ("barrier", 17, 4 * 705 * 6, 6, 64),
    ("barrier", 288, 4 * 720 * 6, 6, 16),
    ("barrier", 1152, 4 * 176 * 6, 6, 4),
    ("barrier", 4608, 4 * 40 * 3, 3, 1),
    ("barrier", 1152, 6496, 1, 8),
    ("rounds_barrier", 17, 4 * 705 * 6, 6, 64),
    ("rounds_barrier", 288, 4 * 720 * 6, 6, 32),
    ("rounds_barrier", 1152, 4 * 176 * 6, 6, 8),
    ("rounds_barrier", 4608, 4 * 40 * 3, 3, 4),
    ("rounds_barrier", 2304, 5, 5, 1),
])
def test_chunk_at_a_barrier(exec, p, m, b, quanta, capfd):
    need_gpu()
    err = _call(p, m, "int32", exec, b, 0, capfd)
    assert f" level_chunk_quanta={quanta} " in err, err


# pieces of 256 quanta at a grid barrier, and with 4-byte lanes from 2^21
# quanta of all ranks' blocks on; else 128
@pytest.mark.parametrize("exec,p,m,dtype,b,piece", [
    ("rounds", 7, 1 << 16, "int32", 4, 128),
    ("rounds_barrier", 7, 1 << 16, "int32", 4, 256),
    ("rounds_barrier", 40, 4 * 255 * 3, "int32", 3, 256),
    ("rounds_barrier", 41, 4 * 257 * 3, "int32", 3, 256),
    ("rounds_barrier", 41, 513 * 3, "u32mat2x2", 3, 256),
    ("rounds_barrier", 101, 1027, "float32", 2, 256),
    ("rounds", 64, 3 * 32767 + 1, "float32", 3, 256),
    ("rounds", 64, 3 * 32767, "float32", 3, 128),
    ("rounds", 101, 3 * 20801, "float32", 3, 256),
])
def test_down_piece(exec, p, m, dtype, b, piece, capfd):
    need_gpu()
    err = _call(p, m, dtype, exec, b, 1, capfd)
    assert f" down_piece={piece} " in err, err


# ranks per down-step item at a barrier: 32, 64 from 2^18 quanta of all ranks'
# blocks on (lines of 8 quanta)
@pytest.mark.parametrize("exec,p,m,ranks", [
    ("rounds", 64, 4 * 4096 * 2, 16),
    ("rounds_barrier", 64, 4 * 4088 * 2, 32),
    ("rounds_barrier", 64, 4 * 4096 * 2, 64),
])
def test_down_ranks(exec, p, m, ranks, capfd):
    need_gpu()
    err = _call(p, m, "int32", exec, 2, 0, capfd)
    assert f" down_ranks={ranks} " in err, err


# more than one 1 KB chunk per CU: 256 threads while two workgroups fit a CU
# by LDS (80 groups), else 512; launch per round counts one round's items
@pytest.mark.parametrize("p,m,exec,b,threads", [
    (300, 65540, "split", 1, 256),
    (320, 65540, "split", 1, 256),
    (576, 65540, "split", 1, 256),
    (640, 65540, "split", 1, 512),
    (320, 400 * 256, "launch", 8, 1024),
])
def test_threads(p, m, exec, b, threads, capfd):
    need_gpu()
    err = _call(p, m, "int32", exec, b, 0, capfd)
    assert f" level_chunk_quanta=64 threads={threads} " in err or \
        exec == "launch" and f" threads={threads} " in err, err


# subtree items: walks, fused under AUTO, where LDS halves the level item's
# chunk and only the level items outnumber the CUs, on rows on the lines; with
# more than one item per CU split from 320 ranks on
@pytest.mark.parametrize("p,m,exec,pad,shown", [
    (1300, 32768, "auto", 0, ("exec=split ", " kernel=level")),
    (1300, 32772, "auto", 28, ("exec=one_launch_fused ", " kernel=subtree")),
    (1300, 32772, "split", 28, ("exec=split ", " kernel=subtree")),
    (1300, 32772, "auto", 29, ("exec=split ", " kernel=level")),
    (1300, 65536, "auto", 0, ("exec=one_launch_fused ", " kernel=subtree")),
    (1300, 65540, "auto", 28, ("exec=split ", " kernel=level")),
    (1152, 32800, "auto", 0, ("exec=split ", " kernel=level")),
    (2600, 32800, "auto", 0, ("exec=split ", " kernel=level")),
    (319, 65568, "auto", 0, ("exec=one_launch_fused ", " kernel=level")),
    (320, 65536, "auto", 0, ("exec=one_launch_fused ", " kernel=level")),
    (320, 65568, "auto", 0, ("exec=split ", " kernel=level")),
    (320, 65568, "auto", 1, ("exec=one_launch_fused ", " kernel=level")),
])
def test_subtree_route(p, m, exec, pad, shown, capfd):
    need_gpu()
    err = _call(p, m, "int32", exec, 1, pad, capfd)
    assert all(w in err for w in shown), err
