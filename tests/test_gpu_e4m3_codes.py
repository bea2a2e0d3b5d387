"""Every E4M3 code through every kernel that reads such pools: where all visible rows are the same row,
the output is its V and the lse one element of its K plus the logarithm of their number, whatever the
arithmetic in between."""
import numpy as np
import pytest
import torch

import paper_2502_13575_amd as ets

pytestmark = pytest.mark.gpu

VS = 0.0217


def values_of(codes):
    return torch.from_numpy(codes).view(torch.float8_e4m3fn).to(torch.float64).numpy()


# leaf queries (4 query heads per kv head), rows: one wave's and a workgroup's items of 16 query rows, one to
# four row blocks, the group kernel's items of 128, the wide kernel's of 256
@pytest.mark.parametrize("d,n,rows,options", [
    (d, n, rows, options) for d in (128, 64) for n, rows, options in [
        (4, 1, {}), (4, 90, {"wave_items": 0}), (8, 100, {}), (16, 97, {}), (64, 130, {}), (200, 16500, {}),
        (64, 129, {"wide_rows": 64}), ("prefill", 1, {}), ("prefill", 100, {})]
    if d == 128 or (n != "prefill" and not options.get("wide_rows"))])
def test_equal_rows_give_their_codes(d, n, rows, options):
    prefill, n = n == "prefill", 32 if n == "prefill" else n
    hkv = 256 // d
    hq = 4 * hkv
    v = np.arange(256, dtype=np.uint8).reshape(hkv, d)         # every code, the two NaNs too
    k = np.where((v & 0x7F) == 0x7F, 0x38, v).astype(np.uint8)  # every number
    kd, vd = (torch.from_numpy(x)[:, None].repeat(1, rows + 1, 1).to("cuda:0") for x in (k, v))
    if prefill:  # duplicated queries of a one-token step below the shared rows
        parent, offset = np.array([-1, 0], np.int32), np.array([0, rows], np.int64)
        tokens, leaves, seen = np.array([rows, 1], np.int32), np.ones(n, np.int32), rows + 1
    else:
        parent, offset = np.array([-1], np.int32), np.array([0], np.int64)
        tokens, leaves, seen = np.array([rows], np.int32), np.zeros(n, np.int32), rows
    # query row r of a kv head asks for K's element r, in turn
    ask = (np.arange(n)[:, None] * 4 + np.arange(4)) % d
    q = np.zeros((n, hkv, 4, d), np.float32)
    np.put_along_axis(q, np.broadcast_to(ask[:, None, :, None], (n, hkv, 4, 1)), 1.0, axis=3)
    qd = torch.from_numpy(q.reshape(n, hq, d)).to("cuda:0").to(torch.bfloat16)
    out = torch.full((n, hq, d), float("nan"), device="cuda:0")
    lse = torch.full((n, hq), float("nan"), device="cuda:0")
    print("case e4m3 codes", d, n, rows, options, prefill, flush=True)
    with ets.Context(hkv, hq, d, ets.ETS_BF16, 0) as ctx:
        for key, value in options.items():
            ctx.set_option(key, value)
        ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, 1.0, VS)
        if prefill:
            ctx.plan_prefill(parent, offset, tokens, leaves)
            ctx.prefill(kd, vd, rows + 1, qd, out, lse)
        else:
            st = ctx.plan(parent, offset, tokens, leaves)
            if rows > 1:
                assert (st.wide_tokens if "wide_rows" in options else st.cascade_tokens) == rows
            # the group kernel; none beside the wide kernel
            assert ctx.item_rows() == (128 if n == 200 else 0 if "wide_rows" in options else 64)
            ws = torch.empty(max(st.workspace_bytes, 16), dtype=torch.uint8, device="cuda:0")
            ctx.decode(kd, vd, rows + 1, qd, out, lse, ws, ws.numel())
        torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(n, hkv, 4, d).astype(np.float64)
    want = np.broadcast_to((values_of(v) * float(np.float32(VS)))[None, :, None], got.shape)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    fin = ~np.isnan(want)
    # fp32: scores in base 2 reach 448 / 8 * log2(e) = 81, and a weight is 2 to the power of their rounding;
    # one rounding per step of 32 rows in the sum of weights, a few in the scale and the quotient
    eps = (96 + seen / 32) * 2.0 ** -24
    assert np.all(np.abs(got - want)[fin] <= eps * np.abs(want)[fin])
    want_lse = values_of(k)[:, ask].transpose(1, 0, 2) / np.sqrt(d) + np.log(seen)
    got_lse = lse.cpu().numpy().reshape(n, hkv, 4)
    assert np.all(np.abs(got_lse - want_lse) <= eps + 8 * 2.0 ** -24 * np.abs(want_lse))
