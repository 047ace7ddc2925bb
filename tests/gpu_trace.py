"""What a call does on the GPU: its kernels and copies, from torch's profiler."""
import json
import os
import tempfile


def trace(call):
    """(kernel names, bytes of the copies to the host, bytes of those to the
    device) of everything that call() puts on the GPU."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as prof:
        call()
        torch.cuda.synchronize()
    with tempfile.TemporaryDirectory() as tmp:
        path = os.path.join(tmp, "trace.json")
        prof.export_chrome_trace(path)
        with open(path) as f:
            events = json.load(f)["traceEvents"]
    kernels = [e["name"] for e in events if e.get("cat") == "kernel"]
    copies = [(e["name"], int(e["args"]["bytes"])) for e in events if e.get("cat") == "gpu_memcpy"]
    return (kernels, sum(n for name, n in copies if "DtoH" in name), sum(n for name, n in copies if "HtoD" in name))
