"""The permutation around the sizes where its kernels and the length of a wave's segment change, against a stable sort."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# pairs of the single-workgroup kernels (segments of 64, 128, 256), of two launches with segments of 64 to 512, of three launches
SIZES = [1, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 4161, 8192, 16384, 16385, 32769, 65536, 131073, 300001]


@pytest.mark.parametrize("Ne", [1, 24, 64, 256])
@pytest.mark.parametrize("skewed", [False, True])
def test_permutation_sizes(Ne, skewed):
    import paper_2604_23108_amd as M
    gen = torch.Generator(device="cuda").manual_seed(Ne)
    for T in SIZES:
        cfg = M.Config(T=T, d=64, n_groups=1, experts_per_group=Ne, d_ff=(64,), k_groups=1, k_experts=1,
                       select_mode=M.SELECT_GLOBAL, dtype=M.BF16)
        e = torch.randint(0, Ne, (T, 1), generator=gen, device="cuda", dtype=torch.int32)
        if skewed:
            e = torch.where(torch.rand((T, 1), generator=gen, device="cuda") < 0.9, Ne // 2, e).int()
        new = lambda n: torch.full((n,), -1, dtype=torch.int32, device="cuda")
        counts, offsets, perm, inv = new(Ne), new(Ne + 1), new(T), new(T)
        ws = torch.empty(M.mohge_workspace_size(cfg, M.CALL_PERMUTE), dtype=torch.uint8, device="cuda")
        print(f"[permute] Ne={Ne} P={T} skewed={skewed}", flush=True)
        M.mohge_permute(cfg, e, counts, offsets, perm, inv, None, None, ws)
        flat = e.flatten().long()
        want = torch.argsort(flat, stable=True)
        assert torch.equal(perm.long(), want)
        assert torch.equal(inv.long()[want], torch.arange(T, device="cuda"))
        assert torch.equal(counts.long(), torch.bincount(flat, minlength=Ne))
        assert torch.equal(offsets[1:].long(), counts.long().cumsum(0)) and offsets[0] == 0


@pytest.mark.parametrize("Ne", [24, 64, 256])
def test_permutation_in_a_workspace_of_another_size(Ne):
    """One workspace sized for the largest batch, and one with room for the counts of segments of 512 pairs only."""
    import paper_2604_23108_amd as M
    gen = torch.Generator(device="cuda").manual_seed(Ne)
    config = lambda T: M.Config(T=T, d=64, n_groups=1, experts_per_group=Ne, d_ff=(64,), k_groups=1, k_experts=1,
                                select_mode=M.SELECT_GLOBAL, dtype=M.BF16)
    sizes = [16385, 16384, 12000, 8192, 4097, 4096, 1000, 64]
    large = torch.empty(M.mohge_workspace_size(config(sizes[0]), M.CALL_PERMUTE), dtype=torch.uint8, device="cuda")
    for T in sizes:
        e = torch.randint(0, Ne, (T, 1), generator=gen, device="cuda", dtype=torch.int32)
        want = torch.argsort(e.flatten().long(), stable=True)
        least = (4 * Ne * -(-T // 512) + 255) // 256 * 256
        for ws in (large, torch.empty(least, dtype=torch.uint8, device="cuda")):
            new = lambda n: torch.full((n,), -1, dtype=torch.int32, device="cuda")
            counts, offsets, perm, inv = new(Ne), new(Ne + 1), new(T), new(T)
            print(f"[permute] Ne={Ne} P={T} workspace={ws.numel()}", flush=True)
            M.mohge_permute(config(T), e, counts, offsets, perm, inv, None, None, ws)
            assert torch.equal(perm.long(), want)
