"""The Python binding's use of torch (no GPU needed)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import torch
for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
import paper_2606_14598_amd as w8a8
class Stream:
    cuda_stream = 4242
torch.cuda.current_stream = lambda index=None: Stream if index == 3 else None
calls = []
w8a8._current_device = lambda: 3
w8a8._call = lambda name, *args: calls.append((name, args))
w8a8._launch(torch.device("cuda", 3), "f", 1, 2)
assert calls == [("f", (1, 2, 4242))], calls
"""


def test_launch_on_a_torch_without_the_internal_accessors():
    subprocess.run([sys.executable, "-c", CODE], check=True, cwd=ROOT)
