"""Selection of images of more than 1024 tokens, on keys that steer each of its
branches, against the oracle on the same keys (whole numbers, so exact)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda"


def keys_of(shape, n, rng):
    """(Stage I, Stage II) keys of one image."""
    smooth = rng.standard_normal(n).astype(np.float32), rng.uniform(-1, 1, n).astype(np.float32)
    if shape == "smooth":
        return smooth
    if shape == "padded":        # a third of the tokens tie at zero in both keys
        pad = rng.random(n) < 0.34
        return np.where(pad, np.float32(0), np.abs(smooth[0])), np.where(pad, np.float32(0), 0.9 + 0.1 * smooth[1])
    if shape == "clusters":      # two narrow clusters far apart and a few outliers
        k = [np.where(rng.random(n) < 0.5, 1e-6, 1e3).astype(np.float32) * (1 + 1e-4 * s) for s in smooth]
        for v in k:
            v[rng.integers(0, n, 5)] = [-3e38, 3e38, 0.0, -1e-40, 7.0]
        return tuple(v.astype(np.float32) for v in k)
    if shape == "period":        # values repeat with the samples' spacing
        i = np.arange(n)
        return (i % 64).astype(np.float32), ((i * 256 // n) % 2 + 1e-3 * (i % 576)).astype(np.float32)
    if shape == "blank":         # every key of both kinds is equal (seven images of ten)
        return (np.full(n, 0.25, np.float32), np.full(n, -0.0, np.float32)) if rng.random() < 0.7 else smooth
    if shape == "one_s":         # every Stage II key is equal
        return smooth[0], np.full(n, 0.5, np.float32)
    assert shape == "sorted"     # ascending and descending
    return np.linspace(1, 2, n, dtype=np.float32), np.linspace(1, -1, n, dtype=np.float32)


# one image up to the sizes at which the loads, the list's place and the sharing
# change; then batches whose shared images (4096 remaining tokens or more, at every
# lambda) get 64, 16, 8, 2 workgroups and one of 256 compute units, and ragged ones
CASES = [([n], share) for n, share in
         [(1025, 0.3), (4095, 0.2), (4097, 0.001), (4608, 0.4), (8191, 0.3), (8193, 0.02), (10240, 0.5), (10241, 0.9),
          (18432, 0.0625), (18796, 0.01)]]
CASES += [([9000] * b, 0.05) for b in (4, 12, 24, 100, 130)]
CASES += [([5000] * 4, 0.1), ([9001, 64, 1, 4200, 1024, 1025, 16384] * 2, 0.11), ([4500] * 40, 0.2), ([17000] * 129, 0.05)]


@pytest.mark.parametrize("shape", ["smooth", "padded", "clusters", "period", "sorted", "blank", "one_s"])
@pytest.mark.parametrize("lam", [0.0, 1 / 3, 0.9, 1.0])
def test_large_images_on_shaped_keys(shape, lam):
    import paper_2607_13500_amd as tr
    rng = np.random.default_rng(3)
    for ci, (N, share) in enumerate(CASES):
        print("[case]", shape, lam, len(N), N[0], share, flush=True)
        K = [max(1, int(share * n)) for n in N]
        made = [keys_of(shape, n, rng) for n in N]
        ki, ks = (torch.from_numpy(np.concatenate([m[j] for m in made])).to(DEV) for j in (0, 1))
        r = tr.Reducer(8, 8, torch.bfloat16, lam=lam, max_images=len(N), max_tokens=sum(N), max_N=max(N),
                       stride_real=ci % 2 == 1)
        idx, src = r.select(ki, ks, N, K)
        idx, src = idx.cpu().numpy(), src.cpu().numpy()
        o = 0
        for b, (n, k) in enumerate(zip(N, K)):
            if b < 16:
                wi, ws = oracle.select(-made[b][0].astype(np.float64), made[b][1].astype(np.float64), k, lam,
                                       stride_mode=ci % 2)
                assert np.array_equal(idx[o:o + k], wi) and np.array_equal(src[o:o + k], ws), (shape, lam, N[:3], b)
            o += k
        r.close()


def test_blank_clip_leaves_nothing_for_the_next_call():
    """A blank image that several workgroups share, then another one in the same
    context: the bitmaps they share are clear again."""
    import paper_2607_13500_amd as tr
    rng = np.random.default_rng(5)
    N, K, lam = [18432, 9000], [1152, 700], 1 / 3
    r = tr.Reducer(8, 8, torch.bfloat16, lam=lam, max_images=2, max_tokens=sum(N), max_N=max(N))
    for shape in ("blank", "smooth", "blank", "one_s", "smooth"):
        made = [keys_of(shape, n, rng) for n in N]
        if shape == "blank":
            made = [(np.ones(n, np.float32), np.ones(n, np.float32)) for n in N]
        ki, ks = (torch.from_numpy(np.concatenate([m[j] for m in made])).to(DEV) for j in (0, 1))
        idx, src = (t.cpu().numpy() for t in r.select(ki, ks, N, K))
        o = 0
        for (n, k), m in zip(zip(N, K), made):
            wi, ws = oracle.select(-m[0].astype(np.float64), m[1].astype(np.float64), k, lam)
            assert np.array_equal(idx[o:o + k], wi) and np.array_equal(src[o:o + k], ws), (shape, n)
            o += k
    r.close()
