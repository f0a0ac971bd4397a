"""Decoding with a second plane: lists and sizes around the limits of the kernel's rules (when the first round is written
ahead of the tables, how much of the list is requested with it) and salient rows at the ends, against float64."""

import numpy as np
import pytest
import torch

from fb4_inputs import DEFAULT_FORMATBOOK, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("block", [32, 16])
@pytest.mark.parametrize("rows,cols,n_sal", [(1, 32, 1), (7, 64, 1), (8, 64, 1), (64, 96, 8), (64, 96, 9), (600, 1152, 75), (600, 1152, 600),
                                             (20000, 320, 2048), (20000, 320, 2049), (20000, 320, 2500), (20000, 320, 2501), (65536, 32, 9000)])
def test_dequantize_with_a_second_plane(rows, cols, n_sal, block, f32):
    check(rows, cols, n_sal, block, f32)


@pytest.mark.parametrize("block", [32, 16])
@pytest.mark.parametrize("rows,cols,n_sal", [(61440, 512, 1), (61440, 512, 2048), (61440, 512, 7680), (61440, 512, 7681), (61439, 512, 2049),
                                             (20000, 1600, 2049), (20000, 1600, 2501)])
def test_dequantize_of_as_many_rounds_as_write_the_first_one_early(rows, cols, n_sal, block):
    # (2.5 rounds of 768 workgroups x 512 threads x 4 words of 8 elements are 61440 x 512)
    check(rows, cols, n_sal, block, False)


def check(rows, cols, n_sal, block, f32):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02883_amd as F
    rng = np.random.default_rng(rows + n_sal)
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    plane = lambda n, e: (rng.integers(0, 256, size=(n, cols // 2)).astype(np.uint8),
                          (rng.integers(0, 33, size=(n, cols // block)) | (rng.integers(e, e + 6, size=(n, cols // block)) << 8)).astype(np.uint16))
    c1, m1 = plane(rows, 124)
    c2, m2 = plane(n_sal, 118)
    sal = np.sort(rng.choice(rows, size=n_sal, replace=False)).astype(np.int32)
    sal[0], sal[-1] = (0, rows - 1) if n_sal > 1 else (rows - 1, rows - 1)
    stride = cols + 8 * (rows % 3)
    out = torch.full((rows, stride), -3.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    dev = lambda a: torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).cuda()
    F.fb4_dequantize(luts, dev(c1), dev(m1), block=block, codes2=dev(c2), meta2=dev(m2), salient_rows=dev(sal), out=out[:, :cols],
                     out_dtype=F.DTYPE_F32 if f32 else F.DTYPE_BF16)
    torch.cuda.synchronize()
    assert (out[:, cols:] == -3.0).all()
    # in float64: integers times powers of two and one sum, exact; then one rounding to the output's type
    table = np.concatenate([DEFAULT_FORMATBOOK.astype(np.float64), np.zeros((1, 8))])

    def decode(c, m):
        nib = np.stack([c & 15, c >> 4], axis=2).reshape(c.shape[0], cols)
        w = np.repeat(m, block, axis=1)
        v = np.ldexp(table[np.minimum(w & 0xFF, 32), nib & 7], (w >> 8).astype(np.int64) - 130)
        return np.where(nib & 8, -v, v)

    ref = decode(c1, m1)
    ref[sal] += decode(c2, m2)
    want = torch.from_numpy(ref).float()
    assert torch.equal(want.double(), torch.from_numpy(ref))      # (the sums are exact in fp32)
    got = out[:, :cols].cpu()
    assert torch.equal(got, want if f32 else want.bfloat16())
    luts.free()
