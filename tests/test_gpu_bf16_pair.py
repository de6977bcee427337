"""Two BF16 increments rounded as a pair (bf16_increment2: packed conversion and
byte selects) against each rounded alone (bf16_increment), bit for bit, on the
kernels' own functions: every upper half of a finite FP32 difference (both signs,
zeros, subnormals, values that round up to infinity) with lower halves below, at and
beyond a tie, every sign beside every other in the pair, and differences of
non-zero states."""
import ctypes as C

import numpy as np
import pytest

from paper_2308_06196_amd import build

pytestmark = pytest.mark.gpu


def test_pair_equals_singles():
    import torch

    print("[case] bf16 pair", flush=True)
    L = C.CDLL(build.build_checks(only_missing=True))
    high = np.arange(1 << 16, dtype=np.uint32)
    high = high[(high & 0x7F80) != 0x7F80]  # finite
    low = np.array([0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF], dtype=np.uint32)
    d = ((high[:, None] << 16) | low[None]).ravel().view(np.float32)
    rng = np.random.default_rng(2)
    pairs = [np.column_stack([d, p]) for p in (d[::-1], -d, rng.permutation(d))]
    o = np.concatenate(pairs).astype(np.float32)
    base = np.zeros_like(o)
    b = rng.uniform(0.0, 2.0, (200000, 2)).astype(np.float32)
    b *= np.float32(10.0) ** rng.integers(-30, 3, b.shape).astype(np.float32)
    delta = rng.uniform(-1.0, 1.0, b.shape) * 10.0 ** rng.integers(-8, 1, b.shape)
    o = np.concatenate([o, (b * (1.0 + delta)).astype(np.float32)])
    base = np.concatenate([base, b])
    n = len(o)
    to, tb = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (o, base))
    word, want = (torch.zeros(n, dtype=torch.int32, device="cuda:0") for _ in range(2))
    st, sw = (torch.zeros((n, 2), dtype=torch.float32, device="cuda:0") for _ in range(2))
    ptr = [C.c_void_p(t.data_ptr()) for t in (to, tb, word, want, st, sw)]
    torch.cuda.synchronize()
    assert L.bf16_pair_check(ptr[0], ptr[1], n, *ptr[2:]) == 0
    assert torch.equal(word, want)
    assert torch.equal(st.view(torch.int32), sw.view(torch.int32))
    # the singles: nearest even for non-negative differences, truncation for the others
    u = (o - base).astype(np.float32).view(np.uint32).astype(np.uint64)
    rne = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) & 0xFFFF
    h = np.where(u & 0x80000000, u >> 16, rne).astype(np.uint32)
    assert np.array_equal(want.cpu().numpy().view(np.uint32), h[:, 0] | h[:, 1] << 16)
