"""The binding's native part (csrc/fastcall.cpp) without a GPU: compiled here with the host's tensors in the place of the
device's, its calls going to Python functions that note their arguments.  Each check runs in a process of its own, so
that a crash of the interpreter is a failed test."""
import os
import subprocess
import sys

import pytest

import paper_2505_07291_amd.build as build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HOST = """
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
namespace c10::hip {
struct HostStream {
    void *stream() const { return nullptr; }
};
inline HostStream host_stream(int) { return {}; }
inline int host_device() { return 0; }
}  // namespace c10::hip
#define is_cuda is_cpu
#define CUDA CPU
#define AutogradCUDA AutogradCPU
#define getCurrentHIPStream host_stream
#define current_device host_device
#include "%s"
"""

PRELUDE = """
import ctypes, sys
sys.path.insert(0, %r)
import torch
import paper_2505_07291_amd as grpo
from importlib import machinery, util
loader = machinery.ExtensionFileLoader("_fastcall", %r)
fast = util.module_from_spec(util.spec_from_loader("_fastcall", loader))
loader.exec_module(fast)
NAMES = ["grpo_workspace_bytes", "grpo_group_advantages", "grpo_logprobs_fwd", "grpo_loss_fwd_bwd", "grpo_loss_aux_fwd_bwd",
         "grpo_total_rewards", "grpo_filter_groups", "grpo_packed_layout"]
calls, keep = [], []
def stub(name):
    f = getattr(grpo.lib(), name)
    if name == "grpo_workspace_bytes":
        return f
    keep.append(ctypes.CFUNCTYPE(ctypes.c_int, *f.argtypes)(lambda *a: calls.append((name,) + a) or 0))
    return keep[-1]
stubs = [stub(n) for n in NAMES]
fast.bind(*[ctypes.cast(s, ctypes.c_void_p).value for s in stubs])
n, v = 6, 24
z = torch.randn(n, v)
tok, old, adv = torch.zeros(n, dtype=torch.int64), torch.zeros(n), torch.ones(n)
ws = torch.empty(grpo.grpo_workspace_bytes(n), dtype=torch.uint8)
ints = torch.ones(n, dtype=torch.int32)
def no_access():
    t = torch.zeros(n)
    torch._C._set_storage_access_error_msg(t, "this tensor's memory is gone")
    return t
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("fastcall")
    src, lib = str(folder / "host.cpp"), str(folder / "_fastcall.so")
    with open(src, "w") as f:
        f.write(HOST % os.path.join(ROOT, "paper_2505_07291_amd", "csrc", "fastcall.cpp"))
    build.compile_fastcall(src, lib)

    def go(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE % (ROOT, lib) + code], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, "status %d\n%s" % (r.returncode, r.stderr[-3000:])
        assert r.stdout.strip().endswith("done"), r.stdout
    return go


def test_a_tensor_whose_memory_cannot_be_had_raises(run):
    """Tensor::data_ptr() throws for such a tensor; with the interpreter's lock released at that point the
    process ended in a segmentation fault."""
    run("""
for call in (lambda bad: fast.total_rewards(bad, ints, ints, 0.1),
             lambda bad: fast.filter_groups(bad, 3),
             lambda bad: fast.group_advantages(bad, 3, 1e-6, 0, None),
             lambda bad: fast.logprobs_fwd(z, tok, None, 1.0, ws) if bad is None else fast.logprobs_fwd(bad[None], tok[:1], None, 1.0, ws),
             lambda bad: fast.loss_fwd_bwd(z, tok, bad, adv, None, 0.2, 0.2, 4.0, 1.0, 0.0, 1.0, z, ws),
             lambda bad: fast.loss_aux_fwd_bwd(z, tok, old, bad, adv, None, None, 0.2, 0.2, 4.0, 1.0, 0.1, 0.1, 0.0, 1.0, z, ws, True)):
    try:
        call(no_access())
    except RuntimeError as e:
        assert "memory is gone" in str(e), e
    else:
        raise AssertionError("no exception")
assert not calls
assert fast.total_rewards(old, ints, ints, 0.1).shape == (n,) and len(calls) == 1  # and the lock is as it was
import threading
t = threading.Thread(target=lambda: fast.total_rewards(old, ints, ints, 0.1))
t.start(), t.join()
assert len(calls) == 2
print("done")
""")


def test_loss_calls_without_a_gradient_tensor_and_in_place(run):
    """The default form of the two loss calls makes the gradient itself, like the logits; in place it is the logits."""
    run("""
from paper_2505_07291_amd import binding
binding._fast = fast
pitched = torch.randn(n, v + 8)[:, :v]
for logits in (z, pitched, pitched[:1], torch.randn(1, 4, v)[0, :1]):
    m = logits.shape[0]
    args = (tok[:m], old[:m])
    for aux in (False, True):
        def call(**kw):
            calls.clear()
            if aux:
                out = grpo.grpo_loss_aux_fwd_bwd(logits, *args, None, adv[:m], kl_coef=0.0, **kw)
            else:
                out = grpo.grpo_loss_fwd_bwd(logits, *args, adv[:m], **kw)
            assert [c[0] for c in calls] == ["grpo_loss_aux_fwd_bwd" if aux else "grpo_loss_fwd_bwd"]
            return out[-1], calls[0]
        at = 23 if aux else 18  # grad_logits among the library's arguments
        grad, sent = call()
        assert grad.shape == logits.shape and grad.stride() == logits.stride() and grad.dtype == logits.dtype
        assert sent[1 + at] == grad.data_ptr() != logits.data_ptr()
        grad, sent = call(workspace=ws)
        assert sent[1 + at] == grad.data_ptr() and sent[2 + at] == ws.data_ptr()
        grad, sent = call(inplace=True)
        assert grad is logits and sent[1 + at] == logits.data_ptr()
        given = torch.empty_strided(logits.shape, logits.stride())
        grad, sent = call(grad_logits=given)
        assert grad is given and sent[1 + at] == given.data_ptr()
        grad, sent = call(grad_logits=given, inplace=True)
        assert grad is logits and sent[1 + at] == logits.data_ptr()
assert fast.loss_fwd_bwd(z, tok, old, adv, None, 0.2, 0.2, 4.0, 1.0, 0.0, 1.0, z.double(), ws) is None
print("done")
""")
