"""How many workgroups a decode launch has: as many as the chip holds of this kernel with this launch's LDS, whatever
contexts the process made before.  In a process of its own: the first context there allows 8 192 requests."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCRIPT = """
import torch
import paper_2410_18248_amd as P

def shares(max_batch, batch, H, Hkv, D, dtype, ctx):
    dev = torch.device("cuda:0")
    td = torch.float32 if dtype == P.LAMPS_F32 else torch.bfloat16
    cfg = P.LampsConfig(1, H, Hkv, D, 16, 1, (ctx + 15) // 16, max_batch, dtype)
    kp = torch.zeros(1, 1, Hkv, 16 * D, dtype=td, device=dev)
    ws = torch.full((P.lamps_workspace_bytes(cfg),), 255, dtype=torch.uint8, device=dev)
    lam = P.Lamps(cfg, kp, kp.clone(), ws)
    table = torch.zeros(batch, (ctx + 15) // 16, dtype=torch.int32, device=dev)
    lens = torch.full((batch,), ctx, dtype=torch.int32, device=dev)
    q = torch.zeros(batch, H, D, dtype=td, device=dev)
    lam.decode_attn(0, batch, q, table, lens, torch.ones(batch, dtype=torch.uint8, device=dev), torch.empty_like(q))
    torch.cuda.synchronize()
    gh = max(g for g in (range(1, 17) if dtype == P.LAMPS_BF16 and H > Hkv else (1, 2, 4)) if H // Hkv % g == 0)
    share = 2 * gh * (D + 2) * 4                     # two slots of a share; records of 16 bytes follow the slots of all
    most = min((64 << 20) // share, 16384) // 4 * 4
    rec = ws[(most * share + 255) // 256 * 256:][:16 * (most + 1)].view(torch.int32).view(-1, 4)
    n = int((rec[:, 3] != -1).sum())
    lam.destroy()
    return n

# bf16, 64 dims, one head a pass: six workgroups on each of 256 CUs, a share for each of their four waves; five in
# the form whose workgroups have a share together
print(shares(8192, 120, 8, 8, 64, P.LAMPS_BF16, 300), shares(120, 120, 8, 8, 64, P.LAMPS_BF16, 300), shares(8192, 40, 8, 8, 64, P.LAMPS_BF16, 300),
      shares(8192, 8192, 1, 1, 64, P.LAMPS_BF16, 40))
# shares of a workgroup: 16 heads of 256 in its LDS, 66 KiB
print(shares(64, 2, 32, 2, 256, P.LAMPS_BF16, 500))
"""


def test_width_is_the_launchs_own():
    out = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr
    got = [[int(x) for x in line.split()] for line in out.stdout.strip().splitlines()]
    assert got[0][:3] == [6144, 6144, 1280]                            # an allowance for many requests takes nothing away
    assert got[0][3] == 4096                                           # many requests do: 32 KiB of lengths, four on a CU
    assert got[1] == [256]
