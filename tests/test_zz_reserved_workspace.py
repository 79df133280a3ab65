"""A workspace reservation that is too small for the splits' partial results (in a process of its own: a reservation holds until the
process ends): prefill linears and decode attention run unsplit with the same results, a call that cannot do without it
returns LPQ_ERR_BUFSIZE and launches nothing, also where only its second launch needs the space."""
import os
import subprocess
import sys

import pytest

CHILD = r"""
import torch
import paper_2403_01136_amd as lpq
g = torch.Generator(device="cuda").manual_seed(5)
lpq.lpq_workspace_reserve(256)
w, x = (torch.randn((512, 4096), generator=g, device="cuda") * 0.02).half(), torch.randn((300, 4096), generator=g, device="cuda").half()
qw = lpq.lpq_quantize_pack(w, 4, 1)
y = lpq.lpq_qlinear_prefill(qw, x)
ref = x.float() @ lpq.lpq_unpack_dequant(qw).t()
assert float((y.float() - ref).norm() / ref.norm()) <= 1e-3, "prefill"
H, d, S, pos = 2, 64, 5056, 5000
one = torch.ones(H * d, dtype=torch.float16, device="cuda")
st = lpq.LayerState(H, d, S, 1, torch.device("cuda"), (one, one), (one, one))
st.k_cache.normal_(generator=g), st.vt_cache.normal_(generator=g)
qkv = torch.randn((1, 3 * H * d), generator=g, device="cuda").half()
out = lpq.lpq_attention(qkv, st, 1, 1, pos - 1)
q = qkv[0, :H * d].view(H, d, 1).double()
p = torch.softmax((st.k_cache[0, :, :pos].double() @ q).squeeze(-1) / d ** 0.5, 1)
ref = (st.vt_cache[0, :, :, :pos].double() @ p.unsqueeze(-1)).reshape(1, -1)
assert float((out.double() - ref).norm() / ref.norm()) <= 1e-3, "attention"
try:
    lpq.lpq_variance_indicator(w, x)
    raise SystemExit("the indicator ran without its workspace")
except lpq.LpqError as e:
    assert e.status == 6, e
torch.cuda.synchronize()
print("reserved ok")
"""


# Two launches of 26 linears: the first needs no workspace, the second (K = 8192 on few rows) splits K and does.
CHILD_REFUSED = r"""
import torch
import paper_2403_01136_amd as lpq
lpq.lpq_workspace_reserve(256)
dev = torch.device("cuda")
def weight(K): return lpq.lpq_quantize_pack(torch.randn((64, K), device=dev).half(), 4, 1)
small, large = weight(128), weight(8192)
layers = [{n: small if i < 7 else large for n in lpq.LINEARS} for i in range(13)]
for M in (8, 20):
    x = {K: torch.randn((M, K), device=dev).half() for K in (128, 8192)}
    xs = [{n: x[layer[n].K] for n in lpq.LINEARS} for layer in layers]
    ys = [{n: torch.full((M, 64), float("nan"), dtype=torch.float16, device=dev) for n in lpq.LINEARS} for _ in layers]
    try:
        lpq.lpq_stage_linears(lpq.Stage(layers, xs, ys), lpq.LPQ_DECODE)
        raise SystemExit("%d rows ran without their workspace" % M)
    except lpq.LpqError as e:
        assert e.status == 6, e
    torch.cuda.synchronize()
    assert all(bool(torch.isnan(y).all()) for d in ys for y in d.values()), "%d rows: a refused call wrote outputs" % M
print("reserved ok")
"""


# Four linears between the two lines of the kernel of few row blocks (1 MiB: the lines at 5.2 and 9.9 MB of codes).
CHILD_LINE = r"""
import sys
import torch
import paper_2403_01136_amd as lpq
dev = torch.device("cuda")
even_share = sys.argv[1] == "even_share"
qw = lpq.lpq_quantize_pack((torch.randn((896, 2048), device=dev) * 0.02).half(), 8, lpq.LPQ_SYM_CHANNEL)
def call(M):
    xs = {n: torch.randn((M, 2048), device=dev).half() for n in lpq.LINEARS}
    ys = {n: torch.empty((M, 896), dtype=torch.float16, device=dev) for n in lpq.LINEARS}
    lpq.lpq_stage_linears(lpq.Stage([{n: qw for n in lpq.LINEARS}], [xs], [ys]), lpq.LPQ_DECODE)
    return lpq.lpq_workspace_bytes()
lpq.lpq_set_decode_routing(0 if even_share else 1, -1)
descs = [(8, lpq.LPQ_SYM_CHANNEL, 2048, 896)] * 4
for M in (24, 43):
    assert lpq.lpq_route_of(descs, lpq.LPQ_DECODE, M)[0] == (lpq.LPQ_ROUTE_EVEN_SHARE if even_share else lpq.LPQ_ROUTE_MID)
assert lpq.lpq_route_of(descs, lpq.LPQ_DECODE, 64)[0] == lpq.LPQ_ROUTE_EVEN_SHARE
if not even_share:
    lpq.lpq_qlinear_decode(qw, torch.randn((24, 2048), device=dev).half())
    assert lpq.lpq_workspace_bytes() <= 8 << 20, "a launch below both lines"
print("bytes", call(24), call(43), call(64))
lpq.lpq_workspace_reserve(1)
for M in (17, 24, 32, 33, 43, 48, 64):
    call(M)
torch.cuda.synchronize()
print("reserved ok")
"""


def run_child(code, *args):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code, *args], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "reserved ok" in r.stdout, r.stdout + r.stderr
    return r.stdout


@pytest.mark.gpu
def test_small_reservation_runs_unsplit():
    run_child(CHILD)


@pytest.mark.gpu
def test_small_reservation_refuses_before_the_first_launch():
    run_child(CHILD_REFUSED)


@pytest.mark.gpu
def test_launches_between_the_lines_ask_for_the_even_share_kernels_workspace():
    """A launch of several linears that goes to the kernel of few row blocks only because of the farther line has the workspace grow as the even-share
    kernel's would: a reservation serves, or refuses, the calls it did, whichever kernel takes them."""
    sizes = [next(line for line in run_child(CHILD_LINE, kernel).splitlines() if line.startswith("bytes")) for kernel in ("mid", "even_share")]
    assert sizes[0] == sizes[1] and int(sizes[0].split()[1]) > 32 << 20, sizes
