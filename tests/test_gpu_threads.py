"""The Python entry points do not keep the interpreter lock while they are inside the library: another thread goes on
while a call allocates or waits for a place in a full launch queue."""
import ctypes
import subprocess
import threading
import time

import pytest
import torch

pytestmark = pytest.mark.gpu

# a cell library whose calls return once another thread has set `go`, or fail after two seconds
SOURCE = """
#include <stddef.h>
#include <time.h>
volatile int entered, go;
size_t ws(int dt, int B, int L, int H, int back) { (void)dt; (void)B; (void)L; (void)H; (void)back; return 256; }
int call(void)
{
    const struct timespec ms = {0, 1000000};
    entered = 1;
    for (int i = 0; i < 2000 && !go; ++i) nanosleep(&ms, 0);
    return go ? 0 : 4;
}
"""


@pytest.fixture(scope="module")
def slow(tmp_path_factory):
    d = tmp_path_factory.mktemp("slow")
    (d / "slow.c").write_text(SOURCE)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(d / "slow.so"), str(d / "slow.c")], check=True)
    return ctypes.CDLL(str(d / "slow.so"))


@pytest.mark.parametrize("entry", ["forward", "backward", "rnn_apply"])
def test_other_threads_run_during_a_call(slow, entry):
    from paper_2510_21450_amd import _host
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    cell = _host.library_cell("slow", 1, 1, address(slow.ws), address(slow.ws), address(slow.call), address(slow.call))
    params, u = torch.zeros(1, 8, device="cuda"), torch.zeros(2, 4, 1, 8, device="cuda")
    flags = [ctypes.c_int.in_dll(slow, n) for n in ("entered", "go")]
    for f in flags:
        f.value = 0
    failed = []

    def work():
        try:
            if entry == "forward":
                _host.forward(cell, params, u, None, 1e-3, 4, False, None, None, None)
            elif entry == "backward":
                _host.backward(cell, params, u, None, u, u, False, None, None, None, None, None)
            else:
                _host.rnn_apply(cell, params, u, None, 1e-3, 4)
        except RuntimeError as e:
            failed.append(str(e))

    t = threading.Thread(target=work)
    t.start()
    while not flags[0].value and t.is_alive():
        time.sleep(0.001)
    flags[1].value = 1
    t.join()
    assert not failed


@pytest.mark.parametrize("anomaly", [False, True])
def test_python_hooks_run_inside_the_calls(anomaly):
    """What calls back into Python from inside (hooks of saved tensors, the stack that anomaly mode records) takes the lock
    itself: same results with and without them, also while another thread keeps the interpreter busy."""
    import paper_2510_21450_amd as P
    B, L, H = 2, 60, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    x, Wx, bias, params, g = rand(B, L, H), rand(3, H, H) / 8, rand(3, H), 0.3 * rand(2, 3, H), rand(B, L, 1, H)

    def grads():
        leaves = [t.clone().requires_grad_() for t in (x, Wx, bias, params)]
        u = P.input_projection_apply(leaves[0], leaves[1], leaves[2], n_heads=1)
        h = P.rnn_apply("gru_diag", leaves[3], u, None, tol=1e-5, max_iter=30)[0]
        y = P.rnn_layer("gru_diag", *leaves, n_heads=1, tol=1e-5, max_iter=30)[0]
        ((h + y) * g).sum().backward()
        return [h.detach(), y.detach(), *(t.grad for t in leaves)]

    want, packed, stop = grads(), [], threading.Event()

    def spin():
        while not stop.is_set():
            sum(range(1000))

    other = threading.Thread(target=spin)
    other.start()
    try:
        with torch.autograd.set_detect_anomaly(anomaly), \
                torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t.shape) or t.cpu(), lambda t: t.cuda()):
            got = grads()
    finally:
        stop.set()
        other.join()
    assert len(packed) >= 8 and all(torch.equal(a, b) for a, b in zip(got, want))
