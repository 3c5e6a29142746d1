"""Which kernels a call takes, by the rules on sizes of the library's host side (compiled for the host alone; nothing is launched)."""
import pytest

from host_routes import P, Routes


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    return Routes(tmp_path_factory.mktemp("routes"))


ONE = ["onepass.sigattn_onepass_plan", "onepass.sigattn_onepass"]


@pytest.mark.parametrize("B,N,H,one", [
    (32, 512, 32, False), (128, 512, 12, True), (127, 512, 12, False),      # heads of two key tiles: 3072 tiles
    (128, 449, 12, True), (128, 448, 12, False),
    (22, 513, 12, True), (21, 513, 12, False),                             # longer ones: 768
    (8, 2048, 12, True), (7, 2048, 12, False), (2, 8192, 12, True),
])
def test_one_pass_where_it_gains(routes, B, N, H, one):
    assert ([l.name for l in routes.bwd(B, N, H, 64)] == ONE) == one
    assert [l.name for l in routes.bwd(B, N, H, 64, workspace=False)] == ["sigattn_bwd_kernel<64>"]


@pytest.mark.parametrize("B,N,H", [(150, 2048, 16), (101, 4096, 16), (9, 16384, 32), (512, 512, 12)])
def test_slices_cover_the_batch_inside_the_workspace(routes, B, N, H):
    need = routes.lib.sigmoid_attn_bwd_onepass_workspace_bytes(B, N, H, 64)
    out, done = routes.bwd(B, N, H, 64), 0
    for plan, work in zip(out[::2], out[1::2]):
        assert [plan.name, work.name] == ONE
        for l in (plan, work):
            assert l.q == P + done * N * H * 64 * 2 and l.B == plan.B and 1 <= l.in_order <= l.B    # in_order: the group
            assert (l.part, l.plan, l.flags) == (plan.part, plan.plan, plan.flags)
        tiles = plan.B * H * -(-N // 256)
        assert work.grid == tiles and plan.grid == -(-tiles // 256)
        assert work.part == 2 * P and work.plan - work.part == plan.B * H * -(-N // 64) * 16384
        assert work.flags - work.plan == tiles * 32 and work.flags + tiles * 32 <= 2 * P + need
        done += plan.B
    assert done == B


@pytest.mark.parametrize("B,N,H,d,fwd,bwd", [
    # (kernel, batch order)                                 one tile a head or all workgroups at once: batch order
    (64, 64, 1, 64, ("pair.sigattn_pair<0>", 0), ("pair.sigattn_pair_bwd", 0)),          # ranked in registers
    (65, 64, 1, 64, ("pair.sigattn_pair<0>", 1), ("pair.sigattn_pair_bwd", 1)),
    (128, 64, 1, 64, ("pair.sigattn_pair<0>", 1), ("pair.sigattn_pair_bwd", 1)),
    (128, 128, 1, 64, ("pair.sigattn_pair<0>", 1), ("sigattn_bwd_kernel<64>", 1)),
    (64, 128, 1, 128, ("half128.sigattn_half<0>", 0), ("half128.sigattn_half_bwd", 0)),
    (128, 128, 1, 128, ("half128.sigattn_half<0>", 1), ("half128.sigattn_half_bwd", 1)),
    (256, 128, 1, 128, ("half128.sigattn_half<0>", 1), ("half128.sigattn_half_bwd", 1)),
    (128, 129, 1, 128, ("half128.sigattn_half<0>", 1), ("half128.sigattn_half_bwd", 0)),  # 512 of two tiles a head: longest first
])
def test_small_launches_of_many_sequences(routes, B, N, H, d, fwd, bwd):
    assert [(l.name, l.in_order) for l in routes.fwd(B, N, N, H, d)] == [fwd]
    assert [(l.name, l.in_order) for l in routes.bwd(B, N, H, d)] == [bwd]
    for which, mode in (("dq", 1), ("dkdv", 2)):
        (l,) = routes.half(which, B, N, H, d)
        if "pair" in l.name or "half128" in l.name:
            assert l.name.endswith(f"<{mode}>") and l.in_order == (B > 64)


@pytest.mark.parametrize("B,Lq,Lk,H,pairs", [
    (8, 40, 148, 8, True), (9, 40, 148, 8, False), (5, 64, 128, 16, True), (11, 64, 128, 8, False),     # 256 of about one length
    (64, 128, 128, 1, True), (65, 100, 100, 1, False), (64, 64, 300, 2, False), (16, 200, 400, 1, True), (3, 200, 400, 8, False),
    (3, 64, 512, 16, True), (7, 64, 512, 8, False), (16, 100, 1000, 2, True), (64, 100, 1000, 1, False),   # short ones besides
    (16, 200, 3000, 1, True), (16, 200, 3000, 2, False), (2, 200, 4000, 4, True),
])
def test_pairs_of_both_passes(routes, B, Lq, Lk, H, pairs):
    for a, b in ((Lq, Lk), (Lk, Lq)):
        assert [l.name for l in routes.cross_bwd(B, a, b, H, 64)] == ["pair.sigattn_pair_bwd" if pairs else "sigattn_bwd_kernel<64>"]
