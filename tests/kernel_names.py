"""The walk kernels a call launches, by their template arguments: a test of a
route's records must also know that the route was taken."""
import re


def walk_kernels(call):
    """Runs `call` under torch's profiler; returns its result and the walk kernels
    launched, each as (name, template arguments): walk_kernel <F64, Kahan, adjoint,
    loop>, batch_walk_kernel <F64, Kahan, loop, shared source, uniform key>."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        result = call()
        torch.cuda.synchronize()
    found = [re.search(r"\b((?:batch_)?walk_kernel)<([^>]*)>", e.name) for e in prof.events()]
    return result, [(m.group(1), [{"true": True, "false": False}.get(a, a) for a in m.group(2).replace(" ", "").split(",")])
                    for m in found if m]


def loops(kernels):
    """The stepping loops of those launches: 4 a grid, 12 by levels, 16 more where the grids cover their boxes."""
    return {int(a[3] if name == "walk_kernel" else a[2]) for name, a in kernels}
