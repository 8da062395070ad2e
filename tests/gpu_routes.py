"""Which of the library's kernels a call launched, from the profiler's trace."""
from __future__ import annotations


def kernels(call) -> list[str]:
    """Names of the library's kernels that call() launched, in order, without
    their arguments ("k_nt_dma<256, 256, ...>" and so on)."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    got = []
    for e in sorted(p.events(), key=lambda e: e.time_range.start):
        name = e.name.replace("void ", "")
        if name.startswith("dl::k_"):
            got.append(name[4:].split("(")[0])
    return got


def base(names: list[str]) -> list[str]:
    """The same without template arguments."""
    return [n.split("<")[0] for n in names]
