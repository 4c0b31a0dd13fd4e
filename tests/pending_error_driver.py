"""Run by test_gpu_pending_error.py in a process of its own: the first step
launch of a process, with a HIP error already pending on the thread."""
import ctypes
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import torch  # noqa: E402

from paper_1407_1309_amd import mpdata  # noqa: E402

psi = torch.full((40, 50), 0.5, dtype=torch.float64, device="cuda")
c = [torch.full((41, 50), 0.1, dtype=torch.float64, device="cuda"),
     torch.full((40, 51), 0.1, dtype=torch.float64, device="cuda")]
plan = mpdata.Plan((40, 50), n_iters=2, opts=mpdata.OPT_FCT, bc=int(sys.argv[1]))
torch.cuda.synchronize()
hip_path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
hip = ctypes.CDLL(hip_path)
assert hip.hipGetLastError() == 0
assert hip.hipSetDevice(9999) != 0          # refused by the runtime; leaves the error pending
assert hip.hipPeekAtLastError() != 0
ptr = [ctypes.c_void_p(x.data_ptr()) for x in (psi, *c)]
rc = mpdata.lib().mpdata_step(plan._handle, ptr[0], None, ptr[1], ptr[2], None, 2)
print("RC", rc, "PENDING", int(hip.hipPeekAtLastError() != 0), flush=True)
hip.hipGetLastError()
torch.cuda.synchronize()
rc = mpdata.lib().mpdata_step(plan._handle, ptr[0], None, ptr[1], ptr[2], None, 2)
torch.cuda.synchronize()
print("AFTER", rc, bool(torch.isfinite(psi).all()), flush=True)
