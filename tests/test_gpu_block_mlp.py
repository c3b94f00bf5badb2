"""The layers behind attention in one launch (gpusq_block_mlp_int8) against the three calls that it stands for, each of which is held against the
CPU oracle elsewhere: every output bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import dev, force_kernel, g  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class _Case:
    def __init__(self, g, M, D, H, seed, scales=(0.02, 0.03, 0.02)):
        self.g, self.M, self.D, self.H = g, M, D, H
        r = torch.Generator(device="cuda").manual_seed(seed)
        normal = lambda *shape: torch.randn(shape, generator=r, device="cuda")
        self.Xq = (normal(M, D) * 31).round().clamp(-127, 127).to(torch.int8)
        self.W = [g.prepare_weights(normal(n, k) * 0.05, torch.int8) for n, k in ((D, D), (H, D), (D, H))]
        self.b = [normal(n) * 0.1 for n in (D, H, D)]
        self.s = [dev(np.array([v], np.float32)) for v in scales]

    def buffers(self):
        M, D, H = self.M, self.D, self.H
        f16, i8 = torch.float16, torch.int8
        return [torch.full(shape, 7, dtype=dt, device="cuda") for shape, dt in (((M, D), f16), ((M, D), i8), ((M, H), i8), ((M, D), f16))]

    def three(self, P, Pq, G, Y):
        g, M, D, H, W, b, s = self.g, self.M, self.D, self.H, self.W, self.b, self.s
        g.calls.gpusq_spgemm_int8_codes(self.Xq, W[0]["packed"], s[0], W[0]["w_scale"], b[0], P, Pq, s[1], M, D, D, g.EPI_BIAS)
        g.calls.gpusq_spgemm_int8(Pq, W[1]["packed"], s[1], W[1]["w_scale"], b[1], G, g.I8, s[2], M, H, D, g.EPI_BIAS | g.EPI_GELU)
        g.calls.gpusq_spgemm_int8(G, W[2]["packed"], s[2], W[2]["w_scale"], b[2], Y, g.F16, None, M, D, H, g.EPI_BIAS)
        return P, Pq, G, Y

    def one(self, P, Pq, G, Y):
        g, M, D, H, W, b, s = self.g, self.M, self.D, self.H, self.W, self.b, self.s
        g.calls.gpusq_block_mlp_int8(self.Xq, W[0]["packed"], s[0], W[0]["w_scale"], b[0], P, Pq, s[1], W[1]["packed"], W[1]["w_scale"], b[1], G, s[2],
                                     W[2]["packed"], W[2]["w_scale"], b[2], Y, M, D, H)
        return P, Pq, G, Y


def _same(a, b):
    bits = lambda t: t.view(torch.int16) if t.dtype == torch.float16 else t  # (of a NaN as well)
    return [int((bits(x) != bits(y)).sum()) for x, y in zip(a, b)] == [0, 0, 0, 0]


# one K step to four; a row, a slab and a row more; one to four slabs to a CU, chunks that differ by one, a last slab of one row; wavefronts
# without narrow channels (D 192, 320, 448); half a panel of narrow (64, 192) and hidden (H 64, 832, 1856) codes; fewer units than wavefronts; LDS for two slabs;
# two rounds
SIZES = [(1, 64, 64), (17, 64, 512), (16, 128, 64), (33, 192, 832), (300, 256, 1024), (4096, 192, 768), (4097, 256, 1024), (8193, 384, 1536),
         (12544, 512, 2048), (777, 320, 1280), (5000, 448, 1856), (9000, 512, 4096), (40000, 128, 256), (20001, 448, 448)]


@pytest.mark.parametrize("M,D,H", SIZES)
def test_one_launch_is_the_three(g, force_kernel, M, D, H):
    c = _Case(g, M, D, H, M + D)
    force_kernel(6)
    assert g.lib().gpusq_block_mlp_int8_launches(M, D, H, 0) == 1
    one = c.one(*c.buffers())
    force_kernel(None)
    three = c.three(*c.buffers())
    assert _same(one, three)


# the pairs of K steps and slabs (of the highest chunk, on 256 CUs) that no size above has: 1 step and 2, 3 slabs, 2 and 3, 4, 3 and 2, 4
@pytest.mark.parametrize("M,D,H", [(4097, 128, 256), (8193, 128, 512), (8193, 256, 1024), (12601, 192, 768), (6304, 384, 1536), (12608, 384, 1536)])
def test_one_launch_is_the_three_at_every_height(g, force_kernel, M, D, H):
    test_one_launch_is_the_three(g, force_kernel, M, D, H)


@pytest.mark.parametrize("scales", [(0.0, 0.03, 0.02), (0.02, 0.0, 0.02), (0.02, 0.03, 0.0), (float("inf"), 0.03, 0.02), (0.02, float("nan"), 0.02), (0.02, 0.03, float("inf")),
                                    (-0.02, -0.03, -0.02), (0.02, 1e-40, 0.02), (0.02, 0.03, 1e-40), (1e30, 0.03, 0.02), (0.02, 1e-6, 1e-6)])
@pytest.mark.parametrize("M,D,H", [(100, 192, 768), (70, 448, 448)])
def test_scales_that_are_no_numbers_or_too_small(g, force_kernel, scales, M, D, H):
    c = _Case(g, M, D, H, 5, scales)
    force_kernel(6)
    one = c.one(*c.buffers())
    force_kernel(None)
    assert _same(one, c.three(*c.buffers()))


def test_buffers_that_overlap(g, force_kernel):
    """Codes over attention's, whole or in part, and outputs over each other: as the three calls leave them"""
    M, D, H = 700, 192, 768
    force_kernel(6)
    for first, second in ((0, 0), (0, 64)):
        out = []
        for call in ("one", "three"):
            c = _Case(g, M, D, H, 9)
            both = torch.zeros((M + second, D), dtype=torch.int8, device="cuda")
            both[:M] = c.Xq
            c.Xq = both[:M]
            P, _, G, Y = c.buffers()
            out.append([t.clone() for t in getattr(c, call)(P, both[second:], G, Y)])
        assert _same(*out)
    out = []
    for call in ("one", "three"):
        c = _Case(g, M, D, H, 9)
        P, Pq, G, _ = c.buffers()
        out.append([t.clone() for t in getattr(c, call)(P, Pq, G, P)])
    assert _same(*out)


def test_a_block_in_a_graph(g):
    """EncoderBlockLinears in one launch behind attention, recorded: replays between eager work, each against the eager block"""
    from paper_2305_10727_amd.pipeline import EncoderBlockLinears
    M, D, H = 3000, 256, 1024
    assert g.lib().gpusq_block_mlp_int8_launches(M, D, H, 0) == 1
    r = torch.Generator(device="cuda").manual_seed(3)
    normal = lambda *shape: torch.randn(shape, generator=r, device="cuda")
    block = EncoderBlockLinears(M, D, H, {k: dev(np.array([v], np.float32)) for k, v in dict(x=0.03, qkv=0.02, attn=0.02, h=0.03, g=0.02).items()})
    block.prepare_weights(normal(3 * D, D) * 0.05, normal(D, D) * 0.05, normal(H, D) * 0.05, normal(D, H) * 0.05)
    x, biases = normal(M, D).half(), [normal(n) * 0.1 for n in (3 * D, D, H, D)]
    attention = lambda qkv, out: out.copy_(qkv[:, 2 * D:])
    block.capture(x, biases, attention)
    for _ in range(3):
        x.copy_(normal(M, D).half())
        got = [t.clone() for t in (block.replay(), block.proj.Y, block.fc1.Xq, block.fc1.Y)]
        for t in (block.fc2.Y, block.proj.Y, block.fc1.Xq, block.fc1.Y):
            t.zero_()
        block.forward(x, biases, attention)
        torch.cuda.synchronize()
        assert _same([got[1], got[2], got[3], got[0]], [block.proj.Y, block.fc1.Xq, block.fc1.Y, block.fc2.Y])
