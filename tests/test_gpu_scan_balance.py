"""fp32: the reverse scan is about as long as the forward scan that keeps its tiles (96 us each, 1.01 times).  The reverse scan's chain waits for
the helpers' products in every step, so it has eight helper waves where this forward scan has four; with the chain
wave forming every address anew in each step it takes 109 us."""
import pytest
import torch

import paper_2406_06484_amd as dn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 32)])
def test_fp32_reverse_scan_is_no_longer_than_the_forward_scan(dk, dv):
    B, L, H = 3, 1500, 8
    g = torch.Generator(device="cuda").manual_seed(1)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k = (torch.nn.functional.normalize(randn(B, L, H, dk), dim=-1) for _ in range(2))
    v, d_o, beta = randn(B, L, H, dv), randn(B, L, H, dv), torch.sigmoid(randn(B, L, H))
    saved, best = None, {}
    dn.deltanet_profile_enable(True)
    try:
        for _ in range(4):  # (the first round also warms up)
            for _ in range(10):
                _, _, saved = dn.deltanet_fwd_save(q, k, v, beta, saved=saved)
                dn.deltanet_bwd_saved(q, k, v, beta, d_o, saved)
            torch.cuda.synchronize()
            for name, (ms, n) in dn.deltanet_profile_collect().items():
                key = "fwd" if "k_scan_fwd_save" in name else "bwd" if "k_scan_bwd" in name else None
                if key:
                    best[key] = min(best.get(key, 1e9), ms / n)
    finally:
        dn.deltanet_profile_enable(False)
    print(dk, dv, best, flush=True)
    assert best["bwd"] <= 1.04 * best["fwd"]
