"""wv_cnn_restore's guard and byte kernels at their edges: tile edges that are
and are not multiples of four, one and many bands of rows per tile, in place,
at odd addresses, and tiles on both sides of the guard.  Expected: the
network's own inference output (checked elsewhere), rounded as documented."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,tx,ty", [(4, 3, 2), (7, 5, 3), (30, 2, 2), (64, 3, 2), (256, 2, 1)])
def test_restore_matches_inference(tile, tx, ty):
    from paper_2208_10859_amd import cnn
    nt = tx * ty
    net = cnn.Net(tile * tile * nt)
    rng = np.random.default_rng(tile)
    params = np.concatenate([np.concatenate([rng.normal(0, (2 / (9 * ci)) ** 0.5, co * 9 * ci),
                                             rng.normal(0, 0.02, co)]) for ci, co in cnn.LAYERS])
    net.set_params(params)
    img = rng.integers(0, 256, (nt, 3, tile, tile), dtype=np.uint8)
    img[::2] //= 8                                # dark tiles: smaller corrections
    plane = img.reshape(ty, tx, 3, tile, tile).transpose(0, 3, 1, 4, 2).reshape(ty * tile, tx * tile, 3)
    x = np.zeros((1, ty * tile, tx * tile, 4), np.float32)
    x[0, ..., :3] = plane.astype(np.float32) * np.float32(1 / 255)
    z = torch.zeros(x.shape, device="cuda")
    net.infer(torch.from_numpy(x).to(torch.bfloat16).cuda(), z)
    zt = z.cpu().numpy()[0, ..., :3].reshape(ty, tile, tx, tile, 3).transpose(0, 2, 4, 1, 3).reshape(img.shape)
    mean = np.abs(zt.astype(np.float64)).mean(axis=(1, 2, 3))
    # a guard well between two tiles' means
    order = np.sort(mean)
    gap = np.argmax(np.diff(order))
    guard = float((order[gap] + order[gap + 1]) / 2)
    keep = mean <= guard
    f = img.astype(np.float32) * np.float32(1 / 255)
    want = np.clip(np.rint((f.astype(np.float64) + zt) * 255.0), 0, 255)
    buf = torch.zeros(img.size + 1, dtype=torch.uint8, device="cuda")
    dev = buf[1:].view(img.shape)                 # odd address
    dev.copy_(torch.from_numpy(img))
    out, fell = net.restore(dev, tile, tx, ty, guard)
    again, fell2 = net.restore(dev, tile, tx, ty, guard, out=dev)   # in place
    assert fell == fell2 == int((~keep).sum()) and 0 < fell < nt
    assert torch.equal(out, again)
    got = out.cpu().numpy()
    assert np.array_equal(got[~keep], img[~keep])
    # float32 against float64 may round one value next to a tie differently
    diff = np.abs(got[keep].astype(np.int64) - want[keep])
    assert diff.max() <= 1 and np.mean(diff > 0) < 1e-3
