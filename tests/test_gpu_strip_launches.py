"""GPU parity of launches of the fused downscaler that other tests do not make: four-wave workgroups in
runs of 16 per XCD (a launch of four rounds of them, on a filter without the eight-wave form, whole and
odd lines), and filters whose 16 adjacent outputs span more than the streaming kernels' 256 elements
(tiled by default; batches and set_band refuse them)."""

import numpy as np
import pytest

import synthgen
from oracle import polyphase as pp

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [64, 63])
def test_runs_of_four_wave_workgroups(w):
    c = synthgen.design_taps(2, 3, 14)  # split taps
    f, of = aol.Polyphase(2, 3, c), pp.Filter(2, 3, c)
    n = 4100  # one workgroup a frame
    U = np.stack([synthgen.uniform_frame(i, 40, w) for i in range(41)]).repeat(100, axis=0)
    U[::7] = 255 - U[::7]
    plan = aol.DownscalePlan([(40, w)], f, f)
    runs = plan.schedule(n)["runs"]
    assert runs["waves"] == 4 and runs["workgroups"] >= 4 * 3 * torch.cuda.get_device_properties(0).multi_processor_count
    y = torch.full((n,) + plan.out_shapes[0], 0xA5, dtype=torch.uint8, device="cuda")
    plan.run([torch.from_numpy(U).cuda()], [y])
    torch.cuda.synchronize()
    plan.close()
    np.testing.assert_array_equal(y.cpu().numpy(), pp.downscale_u8(U, of, of))


@pytest.mark.parametrize("p,q,taps", [(1, 20, 8), (1, 32, 16)])
def test_filters_beyond_the_streaming_kernels(p, q, taps):
    c = synthgen.design_taps(p, q, taps)
    f, of = aol.Polyphase(p, q, c), pp.Filter(p, q, c)
    X = np.stack([synthgen.uniform_frame(i, 170, 333, idx=q) for i in range(2)])
    plan = aol.DownscalePlan([(170, 333)], f, f)
    assert plan.schedule(2)["kernel"] == "tiled"
    y = torch.full((2,) + plan.out_shapes[0], 0xA5, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        plan.run([torch.from_numpy(X).cuda()], [y])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(y.cpu().numpy(), pp.downscale_u8(X, of, of))
        with pytest.raises(aol.AolError) as e:
            plan.set_band(0, 16)
        assert e.value.status == aol.AOL_ERR_UNSUPPORTED
    plan.close()
    with pytest.raises(aol.AolError) as e:
        aol.BatchPlan([(170, 333, f, f)])
    assert e.value.status == aol.AOL_ERR_UNSUPPORTED
