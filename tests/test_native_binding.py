"""CPU tests of the native half of the binding: tensors that have no memory of their own are refused with an exception.

They run in a process of their own, with stand-ins for the two device queries, on fake device tensors (no GPU is used)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROLOGUE = """
import torch
torch._C._cuda_getDevice = lambda: 0
torch._C._cuda_getCurrentRawStream = lambda device: 0
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2501_02625_amd import binding
bf, f32, i8 = torch.bfloat16, torch.float32, torch.int8
desc = binding.make_desc(16, 64, 32, 1, f32)
def new(*shape, dtype=bf):
    return torch.empty(shape, dtype=dtype, device="cuda:0")
def new_state():
    return binding.LinearState(new(16, 64, dtype=i8), new(16, dtype=f32), new(32, 64, dtype=i8), new(32, dtype=f32))
"""


def run(body):
    env = dict(os.environ, PYTHONPATH=ROOT, HIP_VISIBLE_DEVICES="")
    r = subprocess.run([sys.executable, "-c", PROLOGUE + body], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
    return r.stdout


def test_a_tensor_without_storage_raises():
    """Inside vmap a tensor has no data pointer: taking it throws, which has to end as a Python exception."""
    out = run("""
with FakeTensorMode():
    st, Y, W, E = new_state(), new(16, 32, dtype=f32), new(32, 64), new(3, 16, 32)
    ws, EX, G = new(1 << 20, dtype=torch.uint8), new(16, 64, dtype=f32), new(32, 64, dtype=f32)
    def forward(x):
        binding.halo_linear_fwd(desc, x, W, state=st, Y=Y)
        return x
    def backward(e):
        binding.halo_linear_bwd(desc, e, st, workspace=ws, EX=EX, G=G)
        return e
    for f, x in ((forward, new(3, 16, 64)), (backward, E)):
        try:
            torch.vmap(f)(x)
        except RuntimeError as e:
            print("refused" if "storage" in str(e) else repr(e))
""")
    assert out.split() == ["refused", "refused"]


def test_an_allocator_is_never_taken_from_a_fake_tensor():
    """A first call under a mode that fakes tensors must not leave its allocator behind: the next call asks for device
    memory (which fails without a device) instead of handing null pointers to the library."""
    out = run("""
with FakeTensorMode():
    X, W = new(16, 64), new(32, 64)
    try:
        binding.halo_linear_fwd(desc, X, W)
    except binding.HaloError as e:
        print(e.status == binding.HALO_EINVAL)      # fake outputs: null pointers
try:
    binding.halo_linear_fwd(desc, X, W)
except Exception as e:
    print(not isinstance(e, binding.HaloError))
""")
    assert out.split() == ["True", "True"]
