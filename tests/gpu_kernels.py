"""Which kernels a call launches (for tests of the rules that choose them)."""
import collections
import re

import torch
from torch.profiler import ProfilerActivity, profile


def kernels(fn) -> collections.Counter:
    """Launches per kernel name (the template's arguments with it, the
    function's without) of one call of fn."""
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    names = collections.Counter()
    for e in p.events():
        m = re.match(r"(?:void )?rtm::(k_\w+(?:<[^(]*>)?)", e.name)
        if m:
            names[m.group(1)] += 1
    assert names, "no kernel seen"
    return names


def named(names, prefix: str) -> int:
    """Launches of the kernels whose name begins with prefix."""
    return sum(n for k, n in names.items() if k.startswith(prefix))
