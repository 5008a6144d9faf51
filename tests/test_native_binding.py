"""The native marshalling of the per-step calls: what it refuses, and that errors of the C ABI arrive as
OscError with the library's code and text."""
import os
import signal
import subprocess
import sys

import pytest
import torch

import paper_2604_12782_amd as osc


def test_refuses_what_is_not_a_row_major_bf16_matrix():
    X = torch.zeros((4, 64), dtype=torch.bfloat16)
    with pytest.raises(TypeError, match="torch tensor"):
        osc.osc_quantize_act([1, 2, 3])
    for bad in (X[0], X.t(), X.float()):
        with pytest.raises(AssertionError, match="2-D bf16"):
            osc.osc_quantize_act(bad)
    with pytest.raises(AssertionError):
        osc.osc_swiglu_quantize_act(X, X[:, :32])
    with pytest.raises(ValueError, match="holds 1 tensors"):
        osc.osc_quantize_act(X, out=(X,))
    with pytest.raises(TypeError):
        osc.osc_dual_gemm(X, X, None, X, 64, "64", 0, out=X)


def test_error_of_a_truth_value_arrives():
    """A flag whose truth value raises (a tensor of several elements): that error, before anything is launched."""
    X = torch.zeros((4, 64), dtype=torch.bfloat16)
    flag = torch.ones(2)
    for call in (lambda: osc.osc_rmsnorm_quantize_act(X, X[0], want_norm=flag), lambda: osc.osc_swiglu_quantize_act(X, X, want_y=flag),
                 lambda: osc.osc_swiglu_quantize_act_fp8(X, X, want_y=flag), lambda: osc.osc_quantize_act_dynamic(X, want_idx=flag)):
        with pytest.raises(RuntimeError, match="ambiguous"):
            call()


def test_asks_torch_before_using_the_device():
    """Before its first use of the device a process asks torch, which refuses in a process forked after the GPU was
    used: that refusal arrives, from the native calls and from the stream of the others.  (In a process of its
    own, where nothing has used the device yet.)"""
    code = """
import torch
import paper_2604_12782_amd as osc
def refuse(): raise RuntimeError("refused by torch")
torch.cuda._lazy_init = refuse
X = torch.zeros((4, 64), dtype=torch.bfloat16)
out = (X, X, None)
for call in (lambda: osc.osc_quantize_act(X, out=out), lambda: osc.osc_dual_gemm(X, X, None, X, 64, 64, 0, out=X),
             lambda: osc.osc_pack_weight(X, None), lambda: osc.osc_swiglu_quantize_act(X, X)):
    try:
        call()
    except RuntimeError as e:
        assert str(e) == "refused by torch", e
    else:
        raise AssertionError("not refused")
print("all refused")
"""
    run = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True,
                         text=True, timeout=300)
    assert run.returncode == 0 and "all refused" in run.stdout, run.stdout + run.stderr


@pytest.mark.gpu
def test_forked_process_is_refused():
    """In a process forked after the GPU was used, torch's refusal arrives before anything touches the device."""
    X = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda")
    out = osc.osc_quantize_act(X)
    torch.cuda.synchronize()
    pid = os.fork()
    if pid == 0:
        status = 1
        try:
            signal.alarm(20)
            refused = 0
            for call in (lambda: osc.osc_quantize_act(X), lambda: osc.osc_quantize_act(X, out=out), osc.binding._stream):
                try:
                    call()
                except RuntimeError as e:
                    refused += "forked subprocess" in str(e)
            status = 0 if refused == 3 else 2
        finally:
            os._exit(status)
    assert os.waitpid(pid, 0)[1] == 0
    assert torch.equal(osc.osc_quantize_act(X)[0], out[0])  # the parent goes on


@pytest.mark.gpu
def test_errors_and_outputs_on_the_device():
    X = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(osc.OscError, match="multiple of 32") as e:
        osc.osc_quantize_act(X[:, :40])
    assert e.value.code == -2
    out = (torch.empty((4, 32), dtype=torch.uint8, device="cuda"), torch.empty(osc.osc_act_scale_bytes(4, 64), dtype=torch.uint8, device="cuda"), None)
    got = osc.osc_quantize_act(X, out=list(out))
    assert got[0] is out[0] and got[1] is out[1] and got[2] is None
    q = osc.osc_quantize_act(X, ldb=8)
    assert q[2].shape == (4, 8) and q[2].dtype == torch.uint16 and int(q[2].to(torch.int32).sum()) == 0
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):  # the current stream is the one that is used
        torch.cuda._sleep(1000000)
        Y = osc.osc_quantize_act(torch.ones((1, 32), dtype=torch.bfloat16, device="cuda"))[1]
    side.synchronize()
    assert int(Y[0]) == 125
