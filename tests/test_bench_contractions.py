"""The benchmark's count of executed matrix work: seven contractions per sub-block in the backward kernel, eight where a call
of head size 128 runs a dV and a dK role (the launch's own rule: three workgroups per row tile, at most 512 of 128 rows
or 1024 of 64 in all)."""
import bench


def test_contractions_follow_the_roles_of_the_launch():
    assert bench.contractions_per_subblock("hdt_fwd_bf16_d128", 128, 4, 128) == 2
    for tile_m, most in ((128, 512), (64, 1024)):
        assert bench.contractions_per_subblock("hdt_bwd_bf16_d128", 128, most // 3, tile_m) == 8
        assert bench.contractions_per_subblock("hdt_bwd_bf16_d128", 128, most // 3 + 1, tile_m) == 7
        assert bench.contractions_per_subblock("hdt_bwd_bf16_d64", 64, 1, tile_m) == 7
