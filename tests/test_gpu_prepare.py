"""Steps of sja_prepare_profiles from a multiple of four segments on: jobs that start and progress points that lie at every
place of a group of four, lengths around a group and around a step of 256 segments, arrays at any 4-byte boundary."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2509_19086_amd as P
    return P.Engine(0)


@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("length", [1, 3, 4, 5, 255, 256, 257, 259, 1025])
def test_places(engine, oracle, length, offset):
    import torch
    rng = np.random.default_rng(length + offset)
    lens = length + np.arange(24) % 5
    seg_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    S = int(seg_off[-1])
    dur, mem = rng.integers(1, 50, size=S).astype(np.int32), rng.integers(0, 900, size=S).astype(np.int32)
    safe = (rng.random(S) < rng.choice([0.2, 1.0])).astype(np.uint8) * 7
    progress = np.minimum(np.arange(24) % 7, lens).astype(np.int32)
    progress[-3:] = lens[-3:]                       # nothing left
    progress[-6:-3] = np.maximum(lens[-6:-3] - 1, 0)
    up = lambda a: torch.cat([torch.zeros(offset, dtype=torch.from_numpy(a).dtype), torch.from_numpy(a)]).cuda()[offset:]
    out = [torch.full((S + offset,), -7, dtype=torch.int32, device="cuda")[offset:] for _ in range(3)]
    engine.ensure_workspace(300, len(lens), S)
    engine.sja_prepare_profiles(torch.from_numpy(seg_off).cuda(), up(dur), up(mem), up(safe), torch.from_numpy(progress).cuda(), *out)
    want = oracle.prepare(seg_off, dur, mem, safe, progress)
    left = np.arange(S) - np.repeat(seg_off[:-1], lens) >= np.repeat(progress, lens)
    for got, x in zip(out, want):
        got = got.cpu().numpy()
        np.testing.assert_array_equal(got[left], x[left])
        assert (got[~left] == -7).all()
    # the atoms, through the replies
    W, C = rng.integers(0, 60 * length, size=300).astype(np.int32), rng.integers(0, 1000, size=300).astype(np.int32)
    cut = torch.empty((300, len(lens)), dtype=torch.int32, device="cuda")
    engine.sja_fit(torch.from_numpy(W).cuda(), torch.from_numpy(C).cuda(), cut, None)
    np.testing.assert_array_equal(cut.cpu().numpy(), oracle.fit(seg_off, dur, mem, safe, progress, W, C, False)[0])
