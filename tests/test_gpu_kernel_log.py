"""The plan line (DPAR_LOG=1) names the kernel that runs beside the work item
that the rules choose, on every route where the two differ and one of each
where they agree."""

import pytest
import torch

from tests._gpu import _Env, env_unit, lib, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,m,exec,unit,chosen,kernel", [
    (7, 1000, "auto", None, "level", "few_ranks"),
    (8, 1 << 20, "auto", None, "wide", "few_ranks"),
    (8, 1 << 20, "auto", "seq", "postorder", "postorder"),
    (8, 1 << 20, "split", None, "wide", "wide"),
    (1152, 16384, "auto", None, "subtree", "level"),
    (1152, 16384, "split", None, "subtree", "level"),
    (1152, 16384, "split", "sub", "subtree", "subtree"),
    (1152, 16384, "ticket", None, "subtree", "subtree"),
    (1152, 1024, "auto", None, "level", "level"),
    (128, 1 << 18, "auto", None, "postorder", "postorder"),
])
def test_line_names_the_kernel(p, m, exec, unit, chosen, kernel, capfd):
    need_gpu()
    dpar = lib()
    x = torch.randint(-1000, 1000, (p, m), dtype=torch.int32, device="cuda")
    y = torch.zeros_like(x)
    s = torch.cuda.current_stream()
    with env_unit(unit), _Env("DPAR_LOG", 1):
        dpar.dpar_allreduce_ex(dpar.rows(x), dpar.rows(y), p, m, "int32",
                               "sum", 0, exec, s)
    dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    assert f"unit={chosen} " in err and f" kernel={kernel}\n" in err, err
    assert bool((y == x.sum(0, dtype=torch.int64).to(torch.int32)).all())
