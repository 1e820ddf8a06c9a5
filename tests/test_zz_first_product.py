"""Which launches a masked call makes: its first product goes out ahead of the token count where the host polls for the count in
pinned memory, and behind it where the count travels in ordinary host memory (its copy would wait for the product) and at
widths that have no such product.  Read off a trace of the device; results and counts are the same in every case."""
import ctypes as C

import numpy as np
import pytest

from paper_2210_03052_amd import inputs as I

pytestmark = pytest.mark.gpu


def _kernels(call):
    """Names of the kernels that `call` launches, in the order of their start."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    call()                       # whatever a first call sets up stays out of the trace
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        call()
        torch.cuda.synchronize()
    ev = [e for e in p.events() if e.device_type == torch.autograd.DeviceType.CUDA]
    return [e.name for e in sorted(ev, key=lambda e: e.time_range.start)]


@pytest.mark.parametrize("H,early", [(768, True), (192, False)])
def test_first_product_goes_ahead_of_a_pinned_count_only(bt, H, early):
    import torch
    lib, wl = bt.load_library(), I.WORKLOADS["layer_b4_s64"]
    L = I.draw_lengths(wl)
    T, B, S = int(L.sum()), wl.B, wl.S
    rng = np.random.default_rng(H)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    w = lambda *s: dev(rng.normal(0, 0.02, s).astype(np.float16))
    layer = bt.Layer({"w_qkv": w(3 * H, H), "b_qkv": w(3 * H), "w_o": w(H, H), "b_o": w(H), "ln0_g": w(H), "ln0_b": w(H),
                      "w_1": w(4 * H, H), "b_1": w(4 * H), "w_2": w(H, 4 * H), "b_2": w(H), "ln1_g": w(H), "ln1_b": w(H),
                      "heads": H // 64})
    lengths, x = dev(L), dev(rng.normal(0, 1, (B, S, H)).astype(np.float16))
    cu = torch.empty(B + 2, dtype=torch.int32, device="cuda")
    tok = torch.empty(B * S, dtype=torch.int32, device="cuda")
    ws = torch.empty(bt.layer_workspace_bytes(layer, B * S, B, S), dtype=torch.uint8, device="cuda")
    pinned, pageable = torch.empty(1, dtype=torch.int32, pin_memory=True), np.empty(1, np.int32)
    outs, ahead = [], []
    for total, at in ((pinned.numpy(), pinned.data_ptr()), (pageable, pageable.ctypes.data)):
        out = torch.full_like(x, 7.0)
        names = _kernels(lambda: lib.bt_encoder_fwd_masked(
            C.byref(layer.desc), 1, None, x.data_ptr(), None, lengths.data_ptr(), B, S, cu.data_ptr(), tok.data_ptr(),
            C.cast(at, C.POINTER(C.c_int32)), out.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream))
        assert any("offsets" in n for n in names) and any("mha" in n for n in names), names
        ahead.append(any("gemm_counted_kernel" in n for n in names))
        outs.append(out)
        assert total[0] == T
    assert ahead == [early, False]
    assert torch.equal(*outs)
