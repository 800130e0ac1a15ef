"""The packed bit-planes, byte for byte, against a numpy packer written from the layout:
word (kb, t, n) holds, for the 32 groups of 4 codes of 128-block kb of column n, the pattern
of bit t (first code = MSB) with its low 3 bits inverted when the MSB is set (Eq. 6).  Sizes
at the edges of the kernel's tasks (64 columns x one block per wavefront, 4 blocks per
workgroup): one column, 63 / 64 / 65, odd block counts; codes outside the format's range
(UINT and BINARY count modulo 2^b, TERNARY is clamped)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_06003_amd as L  # noqa: E402


def planes(codes, bits, ternary, n_pad):
    N, K = codes.shape
    q = np.clip(codes.astype(np.int64), -1, 1) + 1 if ternary else codes.astype(np.int64)
    out = np.zeros((K // 128, bits, n_pad, 4), dtype=np.uint32)
    for t in range(bits):
        b = ((q >> t) & 1).reshape(N, K // 128, 4, 8, 4)
        pat = b[..., 0] * 8 + b[..., 1] * 4 + b[..., 2] * 2 + b[..., 3]
        idx = np.where(pat >= 8, pat ^ 7, pat)
        word = (idx << (4 * np.arange(8))).sum(axis=-1).astype(np.uint32)  # [N, KB, 4]
        out[:, t, :N] = word.transpose(1, 0, 2)
    return out


@pytest.mark.parametrize("wfmt,bits", [(L.WFMT_UINT, 1), (L.WFMT_UINT, 2), (L.WFMT_UINT, 4), (L.WFMT_BINARY, 1),
                                       (L.WFMT_TERNARY, 2)])
@pytest.mark.parametrize("K,N", [(128, 1), (384, 63), (640, 64), (1152, 65), (512, 300)])
def test_planes_byte_for_byte(wfmt, bits, K, N):
    print(f"\n[case] pack wfmt={wfmt} b={bits} K={K} N={N}", flush=True)
    rng = np.random.default_rng([K, N, wfmt, bits])
    ternary = wfmt == L.WFMT_TERNARY
    codes = rng.integers(-128, 128, (N, K)).astype(np.int8) if ternary else rng.integers(0, 256, (N, K)).astype(np.uint8)
    p = L.problem(K, N, bits, wfmt, K)
    scales = torch.rand(N, 1, device="cuda").half()
    zeros = torch.rand(N, 1, device="cuda").half() if wfmt == L.WFMT_UINT else None
    packed = torch.full((L.packed_weight_size(p),), 0xA5, dtype=torch.uint8, device="cuda")
    L.pack_weights(p, torch.from_numpy(codes).cuda(), scales, zeros, packed)
    torch.cuda.synchronize()
    n_pad = (N + 255) // 256 * 256
    want = planes(codes, bits, ternary, n_pad)
    got = packed.cpu().numpy()[:want.nbytes].view(np.uint32).reshape(want.shape)
    assert np.array_equal(got, want)
