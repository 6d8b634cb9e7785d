"""Kernels that load straight into LDS: in the built code every LDS read of a wave has
returned before the barrier behind which another wave may load over what it read."""

import re

from test_ticket_cpu import _functions


def test_reads_return_before_the_barrier(tmp_path):
    funcs = {k: v for k, v in _functions(tmp_path).items()
             if any(re.match(r"(buffer_load_dwordx4 .* lds|global_load_lds)", x) for x in v)}
    assert len(funcs) > 60
    for name, ins in funcs.items():
        reads = False
        for x in ins:
            if x.startswith("ds_read"):
                reads = True
            elif x.startswith("s_waitcnt") and "lgkmcnt(0)" in x:
                reads = False
            elif x.startswith("s_barrier"):
                assert not reads, name
