"""The documented switches that pick or shape a work item reach the call they
are set for, where the library by itself takes the few-rank kernel or level
items over whole chunks; bit for bit against the sum either way."""

import pytest
import torch

from tests._gpu import _Env, env_unit, lib, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,m,name,value,shown", [
    # 240 wide chunks: three rounds of 64, the other 48 in four pieces each
    (8, 4096 * 240, "DPAR_WIDE_ROUND", 64, " items=384 full_items=192"),
    (8, 4096 * 240, "DPAR_WIDE_TAIL", 0, " items=240 full_items=240"),
    (4, 1 << 18, "DPAR_WAVES", 2, "unit=postorder waves=2 "),
    (4, 1 << 12, "DPAR_LEVEL_LOG2T", 3, " level_chunk_quanta=8 "),
    (1152, 16384, "DPAR_SUB_DEEP", 0, " sub_deep=0"),
    (1152, 16384, "DPAR_SUB_DEEP", 1, " sub_deep=1"),
])
def test_switch_reaches_its_call(p, m, name, value, shown, capfd):
    need_gpu()
    dpar = lib()
    x = torch.randint(-1000, 1000, (p, m), dtype=torch.int32, device="cuda")
    y = torch.zeros_like(x)
    s = torch.cuda.current_stream()
    with env_unit(None), _Env("DPAR_LOG", 1), _Env(name, value):
        dpar.dpar_allreduce(dpar.rows(x), dpar.rows(y), p, m, "int32", "sum",
                            0, s)
    dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    assert shown in err and "in_registers" not in err, err
    assert bool((y == x.sum(0, dtype=torch.int64).to(torch.int32)).all())


@pytest.mark.parametrize("p", [6000, 12000])
@pytest.mark.parametrize("exec", ["auto", "split", "launch", "rounds"])
def test_level_item_wherever_its_chunk_fits(p, exec, capfd):
    """A level item needs LDS for p / 8 values, not for p rows."""
    need_gpu()
    dpar = lib()
    x = torch.randint(-1000, 1000, (p, 520), dtype=torch.int32, device="cuda")
    y = torch.zeros_like(x)
    s = torch.cuda.current_stream()
    with env_unit("level"), _Env("DPAR_LOG", 1):
        dpar.dpar_allreduce_ex(dpar.rows(x), dpar.rows(y), p, 520, "int32",
                               "sum", 2, exec, s)
    dpar.dpar_check_status(s)
    err = capfd.readouterr().err
    assert "unit=level " in err and " kernel=level\n" in err, err
    assert bool((y == x.sum(0, dtype=torch.int64).to(torch.int32)).all())
