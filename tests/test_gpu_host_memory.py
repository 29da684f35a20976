"""A call whose host-side lists cannot be allocated reports it; no C++ exception leaves the library."""
import resource

import pytest

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


def test_step_many_without_host_memory():
    ctx = binding.Context()
    arr = (binding.AgzoStepItem * 1)()           # (the lists are allocated before the first item is read)
    with open("/proc/self/statm") as f:
        now = int(f.read().split()[0]) * resource.getpagesize()
    soft, hard = resource.getrlimit(resource.RLIMIT_AS)
    resource.setrlimit(resource.RLIMIT_AS, (now + (4 << 30), hard))
    try:
        rc = ctx.lib.agzo_step_many(ctx.h, arr, 1 << 28, 1, 1e-3, 0.0, 0)
    finally:
        resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
    assert rc == binding.ENOMEM and b"host memory" in ctx.lib.agzo_last_error(ctx.h)
    ctx.check()
