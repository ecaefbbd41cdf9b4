"""Names of the library's kernels that a call launches."""


def kernels_of(torch, call):
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if "CUDA" in str(e.device_type) and "fmm::" in e.name]
