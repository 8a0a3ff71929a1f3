"""Replays of a batch's graph with other buffers: the new addresses reach the
argument blocks in stream order, between the replay before and the one after."""
import numpy as np
import pytest
import torch

from paper_1905_03277_amd import synth, torch_ops

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_bursts", [1, 112, 113, 230])   # address blocks hold 112 bursts
def test_replays_with_other_buffers_bitwise(n_bursts):
    """Two sets of frames, fields, outputs and noise tables in turn, enqueued
    without a wait; every burst of every call equals its own hmfsr_merge."""
    shapes = [(3, 32, 48, 1.0, 16), (2, 48, 32, 2.0, 16), (1, 32, 32, 1.5, 16)]
    sets, wants = [], []
    for k in range(2):
        args, cache = [], {}
        for i in range(n_bursts):
            key = i % 7 if i < n_bursts - 1 else -1      # few distinct bursts; the last one is its own
            if key not in cache:
                n, h, w, s, t = shapes[i % 3]
                b = synth.make_burst(n, h, w, seed=9000 + 100 * k + key, scale=s, tile_size=t)
                d = b.desc.replace(noise_table=torch_ops.noise_table(b.desc, DEV, bins=16, patches=64, seed=k)) \
                    if key % 2 else b.desc
                a = (b.frames.to(DEV), b.motion.to(DEV), d, b.tuning)
                cache[key] = (a, torch_ops.merge(*a).cpu().numpy(), (n, h, w, s, t))
            args.append(cache[key])
        # the same shapes in the same places in both sets
        sets.append([a for a, _, _ in args])
        wants.append([w for _, w, _ in args])
    print("[case] batch of", n_bursts, flush=True)
    calls = [(k, torch_ops.merge_batch(sets[k])) for k in (0, 1, 0, 0, 1)]
    torch.cuda.synchronize()
    for c, (k, outs) in enumerate(calls):
        for i, (o, w) in enumerate(zip(outs, wants[k])):
            np.testing.assert_array_equal(o.cpu().numpy(), w, err_msg=f"call {c}, burst {i}")


def test_other_buffers_refused_under_capture():
    """On a capturing stream a call with other buffers is refused, and the next eager one is right."""
    bs = [synth.make_burst(3, 32, 48, seed=9400 + k) for k in range(2)]
    args = [[(b.frames.to(DEV), b.motion.to(DEV), b.desc, b.tuning)] for b in bs]
    wants = [torch_ops.merge(*a[0]) for a in args]
    outs = [torch.empty_like(w) for w in wants]
    torch_ops.merge_batch(args[0], [outs[0]])
    torch.cuda.synchronize()
    print("[case] capture", flush=True)
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        with pytest.raises(RuntimeError):
            torch_ops.merge_batch(args[1], [outs[1]])
    torch_ops.merge_batch(args[1], [outs[1]])
    torch.cuda.synchronize()
    assert torch.equal(outs[0], wants[0]) and torch.equal(outs[1], wants[1])
