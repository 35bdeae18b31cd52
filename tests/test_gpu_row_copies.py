"""Row gathers byte for byte: rows of whole 16-byte pieces, of pieces with a rest, shorter than one and of odd bytes; pitches and addresses; counts around what a
block and a thread copy; nothing written past a row or past the count."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_09887_amd import binding
    binding.lib()
    return binding


def placed(n, width, pitch, offset, seed):
    """[n, width] bytes `pitch` apart that start `offset` bytes into an allocation, and the allocation."""
    flat = torch.randint(0, 256, (n * pitch + offset,), generator=torch.Generator().manual_seed(seed)).to(torch.uint8).cuda()
    return flat.as_strided((n, width), (pitch, 1), offset), flat


@pytest.mark.parametrize("width,src_pad,dst_pad,offset", [(4, 0, 0, 0), (12, 4, 0, 4), (16, 0, 0, 0), (20, 0, 12, 0), (64, 0, 64, 4), (200, 0, 56, 0), (188, 4, 4, 8), (512, 0, 0, 0),
                                                          (36, 3, 0, 0), (33, 0, 0, 0), (200, 0, 0, 2), (1, 0, 0, 0), (16, 0, 0, 1), (5000, 0, 8, 4)])
@pytest.mark.parametrize("n", [1, 7, 300, 5003])
def test_rows(B, width, src_pad, dst_pad, offset, n):
    src, _ = placed(1009, width, width + src_pad, offset, 1)
    out, flat = placed(n, width, width + dst_pad, offset, 2)
    ids = np.random.default_rng(n).integers(0, 1009, n).astype(np.int32)
    want, kept = src[torch.as_tensor(ids).long().cuda()].clone(), flat.clone()
    B.tma_gather_rows(torch.as_tensor(ids).cuda(), src, out=out)
    assert torch.equal(out, want)
    kept.as_strided(out.shape, out.stride(), offset).copy_(want)
    assert torch.equal(flat, kept)


@pytest.mark.parametrize("count", [0, 1, 130, 300, 999])
def test_count_on_the_device(B, count):
    src, _ = placed(100, 100, 100, 0, 3)
    out, flat = placed(300, 100, 112, 0, 4)
    ids = torch.randint(0, 100, (300,), dtype=torch.int32).cuda()
    n = min(count, 300)
    kept, want = flat.clone(), src[ids[:n].long()].clone()
    B.tma_gather_rows_dev(ids, torch.tensor([count], dtype=torch.int32, device="cuda"), src, out)
    kept.as_strided((300, 100), (112, 1), 0)[:n].copy_(want)
    assert torch.equal(flat, kept)


def test_more_rows_than_a_launch_has_blocks(B):
    n, width = (1 << 24) + 5, 513     # a row alone fills a block
    src, _ = placed(1009, width, width, 0, 5)
    ids = torch.randint(0, 1009, (n,), generator=torch.Generator().manual_seed(6), dtype=torch.int32).cuda()
    out = B.tma_gather_rows(ids, src)
    for at in range(0, n, 1 << 20):
        assert torch.equal(out[at:at + (1 << 20)], src[ids[at:at + (1 << 20)].long()])
