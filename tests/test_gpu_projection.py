"""The projection of the FP8 consumer at the edges of its tiles (256 tokens x
256 features, steps of 64 columns, two ahead) and where the Q features end
inside a tile, below and above the width from which on the pipelined kernel
runs (3072): codes and statistics against the float64 oracle, within the
bands that test_gpu_fp8 derives.  Columns past d hold NaN."""

import numpy as np
import pytest
import torch

from oracle import fp8_consumer
from workloads import WORKLOADS, all_weights

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU machines, skipped there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2602_18851_amd import Spectral  # noqa: E402
from test_gpu_fp8 import check_head, layer_tokens  # noqa: E402

CASES = [
    # (id, d, pad, seq, n_q, n_kv, d_h)
    ("one-column", 1, 7, 2, 1, 1, 16),                 # one ragged step
    ("one-step-one-tile", 64, 0, 256, 6, 2, 32),       # 256 tokens, 192 + 64 features
    ("step-and-a-column", 65, 7, 257, 3, 1, 16),       # 48 + 16 features
    ("two-steps", 128, 8, 128, 12, 3, 32),             # Q ends inside the second tile
    ("three-steps-ragged", 200, 0, 300, 5, 5, 64),     # Q ends at 320: inside a wave's part
    ("four-steps-ragged", 250, 14, 255, 3, 1, 128),    # Q ends at 384, K at 512
    ("last-short", 3071, 1, 130, 2, 1, 64),
    ("long-one-tile", 3072, 0, 256, 6, 2, 32),
    ("long-ragged-step", 3073, 7, 257, 3, 1, 16),
    ("long-odd-steps", 3136, 8, 1, 12, 3, 32),         # 49 steps, one token
    ("long-ragged-even-steps", 3160, 0, 300, 5, 5, 64),
    ("long-three-tiles", 3200, 8, 255, 3, 1, 128),
]


def _nan_padded(t, pad):
    p = torch.full((*t.shape[:-1], t.shape[-1] + pad), float("nan"), dtype=t.dtype)
    p[..., :t.shape[-1]] = t
    return p.cuda()[..., :t.shape[-1]]


@pytest.mark.parametrize("name,d,pad,seq,n_q,n_kv,dh", CASES, ids=[c[0] for c in CASES])
def test_projection_edges(name, d, pad, seq, n_q, n_kv, dh):
    wl = WORKLOADS["llama2-70b-gqa"].replace(key=name, std=0.02, n_layers=2, d_model=d, n_q=n_q, n_kv=n_kv,
                                             head_dim=dh)
    wq, wk = all_weights(wl, "cpu")
    xs = [layer_tokens(wl, seq, l) for l in range(2)]
    scales = [max(np.abs(fp8_consumer.head_logits(xs[l].double().numpy(), wq[l].double().numpy(),
                                                  wk[l].double().numpy(), h, n_kv, dh)).max()
                  for h in range(n_q)) / 470.0 for l in range(2)]
    est = Spectral(2, d, n_q, n_kv, dh, wl.dtype, wl.alpha, ld=d + pad)
    scale = torch.tensor(scales, dtype=torch.float32, device="cuda")
    max_abs, n_over, codes = est.logits_fp8(_nan_padded(torch.stack(xs), pad), _nan_padded(wq, pad),
                                            _nan_padded(wk, pad), scale, want_codes=True)
    torch.cuda.synchronize()
    max_abs, n_over, codes, s32 = (t.cpu().numpy() for t in (max_abs, n_over, codes, scale))
    for l in range(2):
        for h in range(n_q):
            check_head(codes[l, h], max_abs[l, h], n_over[l, h], xs[l], wq[l], wk[l], float(s32[l]), h, n_kv, dh)
