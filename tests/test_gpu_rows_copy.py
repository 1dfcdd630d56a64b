"""Layout copies (dualkv_repack / dualkv_replicate) at the row sizes where their kernels change (31 and 32 units of 4 and 16
bytes, 128 and 129 units), bases that allow only 4-byte units, more sequences than a workgroup copies a prompt row for, empty
sequences and prompts; byte for byte against the oracle's packings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,lens", [(5, [3, 0, 7, 1]), (0, [2, 0, 3]), (3, [0] * 16 + [2]), (130, [1]), (2, [i % 3 for i in range(35)])])
@pytest.mark.parametrize("row_bytes", [4, 16, 124, 128, 496, 512, 516, 2048, 2064, 4128])
@pytest.mark.parametrize("shift", [0, 4])
def test_rows_copy(P, lens, row_bytes, shift):
    import torch
    from oracle import attention_oracle as orc
    from paper_2605_15422_amd import binding as B
    print("case rows", P, len(lens), row_bytes, shift, flush=True)
    N, cu = len(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, w = int(cu[-1]), row_bytes // 4
    x = np.random.default_rng(row_bytes + P).integers(0, 2**31, size=(P + T, w)).astype(np.int32)
    std, _ = orc.replicated_layout(P, cu, x[:P], x[P:])
    cu_dev = torch.from_numpy(cu).cuda()

    def dev(rows, a=None):
        t = torch.full((rows * w + shift // 4 + 8,), -5, dtype=torch.int32, device="cuda")
        v = t[shift // 4:shift // 4 + rows * w]
        if a is not None:
            v.copy_(torch.from_numpy(np.ascontiguousarray(a).reshape(-1)))
        return t, v

    (_, packed), (lt, long_), (bt, back) = dev(P + T, x), dev(N * P + T), dev(P + T)
    pos_l = torch.full((N * P + T,), -1, dtype=torch.int32, device="cuda")
    pos_p = torch.full((P + T,), -1, dtype=torch.int32, device="cuda")
    B.dualkv_replicate(N, P, T, cu_dev, row_bytes, packed, long_, pos_l)
    B.dualkv_repack(N, P, T, cu_dev, row_bytes, long_, back, pos_p)
    assert np.array_equal(long_.cpu().numpy().reshape(-1, w), std)
    assert np.array_equal(back.cpu().numpy().reshape(-1, w), x)
    assert np.array_equal(pos_l.cpu().numpy(), orc.position_ids_replicated(P, cu))
    assert np.array_equal(pos_p.cpu().numpy(), orc.position_ids_single_prompt(P, cu))
    for t in (lt, bt):   # nothing outside the rows is written
        assert (t[:shift // 4] == -5).all() and (t[-(8 if shift == 0 else 7):] == -5).all()


def device_check(N, P, lens, row_bytes, shift=0):
    """Both copies against gathers by torch on the device; 4-byte units where `shift` moves the bases by 4 bytes."""
    import torch
    from paper_2605_15422_amd import binding as B
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, w = int(cu[-1]), row_bytes // 4
    idx = np.concatenate([np.concatenate([np.arange(P), P + np.arange(cu[i], cu[i + 1])]) for i in range(N)])
    cu_dev = torch.from_numpy(cu).cuda()

    def dev(rows):
        return torch.full((rows * w + shift // 4,), -5, dtype=torch.int32, device="cuda")[shift // 4:]

    packed, long_, back = dev(P + T), dev(N * P + T), dev(P + T)
    packed.copy_(torch.randint(0, 2**31 - 1, (packed.numel(),), dtype=torch.int32, device="cuda"))
    B.dualkv_replicate(N, P, T, cu_dev, row_bytes, packed, long_)
    assert torch.equal(long_.view(-1, w), packed.view(-1, w)[torch.from_numpy(idx).cuda()])
    B.dualkv_repack(N, P, T, cu_dev, row_bytes, long_, back)
    assert torch.equal(back, packed)


@pytest.mark.parametrize("units", [255, 256, 257, 511, 513, 768, 769, 1024, 1025, 2305])
@pytest.mark.parametrize("unit_bytes", [4, 16])
def test_long_rows(units, unit_bytes):
    """Around one, two, three and four units of each of the 256 threads of a row."""
    print("case long rows", units, unit_bytes, flush=True)
    device_check(5, 7, [3, 0, 9, 1, 4], units * unit_bytes)
    device_check(3, 2, [1, 40, 0], units * unit_bytes, shift=4)


@pytest.mark.parametrize("P,N", [(8, 35), (40, 14), (36, 35), (75, 35), (130, 35), (260, 17), (4300, 1)])
@pytest.mark.parametrize("row_bytes", [512, 2064])
def test_copies_of_a_prompt_row(P, N, row_bytes):
    """1, 2, 4, 8 and 16 copies per workgroup, sequences that they do not divide, a wave and a workgroup per row."""
    print("case copies", P, N, row_bytes, flush=True)
    device_check(N, P, [i % 3 for i in range(N)], row_bytes)


@pytest.mark.parametrize("shift", [0, 4])
def test_copies_larger_than_the_cache(shift):
    """Source and destination of 160 MB each: the variant that bypasses the caches, in 16- and 4-byte units."""
    print("case large copy", shift, flush=True)
    device_check(4, 4000, [4000, 0, 5000, 7001], 8192, shift)
