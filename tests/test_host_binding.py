"""The binding on a torch without the private stream names."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_stream_handle_without_private_torch_names():
    code = ("import types, torch\n"
            "del torch._C._cuda_getCurrentRawStream\n"
            "from paper_2302_11719_amd import core\n"
            "torch.cuda.current_stream = lambda: types.SimpleNamespace(cuda_stream=1234)\n"
            "assert core._stream() == 1234\n")
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, timeout=120)
