"""A workspace reservation that is too small for the splits' partial results (in a process of its own: a reservation holds until the
process ends): prefill linears and decode attention run unsplit with the same results, a call that cannot do without it
returns LPQ_ERR_BUFSIZE."""
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


@pytest.mark.gpu
def test_small_reservation_runs_unsplit():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "reserved ok" in r.stdout, r.stdout + r.stderr
