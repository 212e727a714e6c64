"""Down-step of the round-structured executors: two neighbouring ranks per
wavefront, siblings sharing one read of their parent's block, in pieces of 128
quanta; every tree layout, odd last levels (a neighbour that is no sibling, a
rank alone), blocks around one and two pieces, unaligned rows, in place; bit
for bit against the oracle."""

import numpy as np
import pytest
import torch

from oracle import c_oracle
from tests._gpu import assert_all_ranks_equal, lib, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,op", [("int32", "max"), ("float32", "sum"),
                                      ("u32mat2x2", "matmul")])
@pytest.mark.parametrize("exec", ["rounds", "rounds_barrier"])
@pytest.mark.parametrize("alg", ["dual", "single", "reduce_bcast"])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6, 8, 11, 13, 40, 101, 300])
def test_every_tree(p, alg, exec, dtype, op):
    need_gpu()
    dpar = lib()
    s = torch.cuda.current_stream()
    r = np.random.default_rng(5100 + p)
    # three blocks of 120, 128, 136, 256 and 264 quanta on 16-byte lanes, and
    # of about 256 on 4-byte ones
    quanta = [360, 384, 408, 768, 792]
    sizes = quanta if op == "matmul" else [4 * q for q in quanta] + [771]
    for m in sizes:
        if dtype == "float32":
            x = r.standard_normal((p, m), np.float32)
        elif dtype == "int32":
            x = r.integers(-1 << 31, 1 << 31, (p, m), dtype=np.int32)
        else:
            x = r.integers(0, 1 << 32, (p, m, 4), dtype=np.uint32)
        want = c_oracle.allreduce(x, dtype, op,
                                  layout="dual" if alg == "dual" else "single",
                                  threads=8)
        flat = np.ascontiguousarray(x).view(np.int32).reshape(p, -1)
        n = flat.shape[1]
        for offset, in_place in ((0, False), (1, True)):
            big = torch.full((p, n + 8), -7, dtype=torch.int32, device="cuda")
            big[:, offset:offset + n] = torch.from_numpy(flat).cuda()
            out = big if in_place else torch.full_like(big, -7)
            dpar.dpar_allreduce_opt(
                dpar.rows(big[:, offset:]), dpar.rows(out[:, offset:]), p, m,
                dtype, op, 3, alg, exec, 0, -1, s)
            dpar.dpar_check_status(s)
            got = out.cpu().numpy()
            assert (got[:, :offset] == -7).all()
            assert (got[:, offset + n:] == -7).all()
            got = np.ascontiguousarray(got[:, offset:offset + n])
            assert_all_ranks_equal(got.view(x.dtype).reshape(x.shape), want,
                                   f"p={p} m={m} {alg} {exec} +{offset}")
