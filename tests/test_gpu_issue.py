"""Short runs of frames in flight issued by one host thread per stream: fewer frames than streams, as many, a few more."""
import pytest

from inputs import build_net, build_sequence
from test_gpu_frames import CASES, in_flight, one_by_one, same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["c3_resnet_96", "c4_hrnet_128x96"])
def test_short_runs_issued_by_one_thread_per_stream(name):
    """The bits of one call per frame, whatever the number of frames of a call and of streams, threads starting and ending
    with every call."""
    cfg, kn, ks = CASES[name]
    net, seq = build_net(cfg, **kn), build_sequence(cfg, **dict(ks, n_frames=14))
    ref = one_by_one(net, seq)
    for depth, cuts in [(4, (3,)), (4, (2, 4, 5)), (3, (3, 4)), (2, (3, 3)), (4, ())]:
        print(f"{name}: depth {depth}, calls {cuts or 'one'}", flush=True)
        same(ref, in_flight(net, seq, depth, 1, cuts), f"depth {depth}, cuts {cuts}")
