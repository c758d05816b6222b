"""What a run call takes as its stream (no GPU: a host-only plan refuses to run only after the stream was taken)."""
import enum
import types

import numpy as np
import pytest

from paper_1901_00041_amd import st_conv as sc


class Handle(int):
    pass


class Named(enum.IntEnum):
    DEFAULT = 0


@pytest.mark.parametrize("stream", [None, 0, Handle(0), Named.DEFAULT, False, types.SimpleNamespace(cuda_stream=0), types.SimpleNamespace(cuda_stream=np.int64(0))])
@pytest.mark.parametrize("run", [sc.st_conv_run, sc.st_conv_run_time_only])
def test_accepted_streams(run, stream):
    desc = sc.make_desc(1, 8, 3, 4, 8, 1, 1, 1, 0, "bf16", "f32", 0x1000, 0x2000, 0x3000)
    plan = sc.st_conv_plan([desc], sc.plan_opts(host_only=1))
    with pytest.raises(sc.StError) as refused:
        run(plan, stream)
    assert refused.value.status == sc.ST_ERR_UNSUPPORTED
