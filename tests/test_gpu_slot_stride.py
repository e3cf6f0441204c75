"""Slot strides of the populations: every stride that is reported can be set,
and the autotuner measures each layout once."""
import numpy as np
import pytest

from gpu_util import say
from paper_1909_13772_amd import inputs, wlb

STRIDES = (16384, 2048, 1028, 0)


def test_every_reported_stride_can_be_set():
    # slots of 69 MiB
    dom = (300, 250, 240)
    h, _ = wlb.wlb_blocks_create(wlb.single_block(dom), dom, (1, 1, 1), 19, wlb.F32)
    try:
        size = wlb.wlb_info(h).pop_bytes
        for kib in STRIDES + (1028, 16384):
            wlb.wlb_set_slot_round(h, kib)
            info = wlb.wlb_info(h)
            assert info.slot_round_kib == kib and info.pop_bytes == size
        for kib in (1, 1024, 1027, 4096, -1):
            with pytest.raises(wlb.WlbError):
                wlb.wlb_set_slot_round(h, kib)
    finally:
        wlb.wlb_blocks_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("dom,storage", [((300, 250, 240), wlb.F32), ((200, 210, 203), wlb.F64), ((168, 160, 157), wlb.F32)])
def test_every_stride_gives_the_same_bits(dom, storage):
    """Slots of 69, 66 and 17 MiB."""
    say(f"case strides {dom} storage {storage}")
    rho, u = inputs.random_state(dom, seed=5, umag=0.01)
    ref = None
    for kib in STRIDES:
        B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=storage)
        try:
            B.set_slot_round(kib)
            B.init(wlb.TRT, wlb.make_params(tau=0.8), rho, u)
            assert B.info().slot_round_kib == kib
            B.step(3)
            got = B.moments()
        finally:
            B.close()
        ref = got if ref is None else ref
        assert all(np.array_equal(a, b) for a, b in zip(got, ref)), kib


@pytest.mark.gpu
@pytest.mark.parametrize("dom,strides", [((168, 160, 157), [0]),  # 17 MiB: 16384 and 1028 are one layout, 2048 and 0 another
                                         ((256, 255, 256), [0, 2048, 1028]),  # 64.75 MiB
                                         ((256, 254, 254), []),  # 64 MiB, a multiple of 16 MiB already
                                         ((64, 50, 50), [])])
def test_autotuner_measures_each_layout_once(dom, strides, monkeypatch, capfd):
    say(f"case tuned strides {dom}")
    monkeypatch.setenv("WLB_AUTOTUNE_LOG", "1")
    rho, u = inputs.uniform_state(dom)
    B = wlb.Blocks(wlb.single_block(dom), dom, (1, 1, 1), stencil=19, storage=wlb.F32)
    try:
        B.init(wlb.TRT, wlb.make_params(tau=0.8, autotune=1), rho, u)
        got = B.info().slot_round_kib
    finally:
        B.close()
    err = capfd.readouterr().err
    tried = [int(line.split("rounding")[1].split("KiB")[0]) for line in err.splitlines() if "slot stride rounding" in line]
    assert tried == strides and got in strides + [16384]
