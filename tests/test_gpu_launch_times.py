"""Times of GEMM launches against other launches on the same GPU: the tile and the splits that the library chooses against
forced ones, and epilogues against each other on one tile.  Nothing here depends on how fast the GPU is; each bound lies
between what was measured on either side of it (the figures at each case)."""
import pytest
import torch

import paper_2002_05645_amd as P
from paper_2002_05645_amd import binding as B

pytestmark = pytest.mark.gpu


class Launches:
    """One set of buffers, and contexts whose accumulating launches run over a given number of K splits (0: the library's)."""

    def __init__(self, monkeypatch):
        self.monkeypatch = monkeypatch
        gen = torch.Generator(device="cuda").manual_seed(0)
        self.a, self.b, self.aux = (torch.randn(1 << 25, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(3))
        self.bias = torch.zeros(1 << 16, device="cuda", dtype=torch.bfloat16)
        self.c = torch.zeros(1 << 24, device="cuda")
        self.stream = torch.cuda.current_stream().cuda_stream
        self.ctxs = {}

    def ctx(self, splits):
        if splits not in self.ctxs:
            self.monkeypatch.setenv("L2L_SPLIT_WS_MB", "64")
            self.monkeypatch.setenv("L2L_FORCE_SPLITS", str(splits))
            self.ctxs[splits] = P.Context(P.make_config(64, 2, 128, 16, 2, 2, "bf16", 1e-5, 0), self.stream)
        return self.ctxs[splits]

    def close(self):
        for c in self.ctxs.values():
            c.close()

    def us(self, kc, M, N, K, out_f32=False, impl=0, splits=0, **kw):
        """shortest of several averages over back-to-back launches, in microseconds"""
        lda, ldb = ((K if kc else M) + 7) // 8 * 8, ((K if kc else N) + 7) // 8 * 8
        assert (M if kc else K) * lda <= self.a.numel() and (N if kc else K) * ldb <= self.b.numel()
        assert M * N <= self.c.numel() and N <= self.bias.numel()
        c = self.ctx(splits)
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = float("inf")
        for _ in range(8):
            begin.record()
            for _ in range(40):
                c.op_gemm_ex(P.L2L_BF16, out_f32, kc, kc, M, N, K, self.a, lda, self.b, ldb, self.c, N, impl=impl, ldr=N, ldaux=N, **kw)
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end) / 40 * 1e3)
        return best


@pytest.fixture
def launches(monkeypatch):
    s = Launches(monkeypatch)
    yield s
    s.close()


@pytest.mark.parametrize("M,N,K", [(4096, 1024, 1024), (3000, 1024, 256)])
@pytest.mark.parametrize("out_f32", [False, True])
def test_scaled_product_takes_no_longer_than_the_plain_one(launches, M, N, K, out_f32):
    # 256 x 256 tiles: through the kernel that reads its flags at run time 1.24 to 1.40 times the plain product's time, with
    # the scaling compiled in 0.99 to 1.01
    scaled, plain = (launches.us(1, M, N, K, out_f32, impl=106, alpha=alpha) for alpha in (0.5, 1.0))
    assert scaled < 1.12 * plain


@pytest.mark.parametrize("flags", ["gelugrad", "bias and residual", "fp32 residual"])
def test_element_wise_epilogue_of_the_two_wave_group_tile(launches, flags):
    # N = 257: rows that allow no 16-byte access.  Against the 256 x 256 tile that stages through registers and goes element by
    # element as well: an element's operands requested one at a time, behind the store before, 1.18, 0.98 and 1.14 times its
    # time; four rows at a time 0.97, 0.45 and 0.85
    kw = {"gelugrad": dict(epi=B.EPI_GELUGRAD, aux=launches.aux), "bias and residual": dict(bias=launches.bias, resid=launches.aux),
          "fp32 residual": dict(out_f32=True, resid=launches.aux)}[flags]
    bound = {"gelugrad": 1.07, "bias and residual": 0.7, "fp32 residual": 1.0}[flags]
    direct, staged = (launches.us(1, 8192, 257, 256, impl=impl, **kw) for impl in (106, 103))
    assert direct < bound * staged


@pytest.mark.parametrize("M,N,K", [(4096, 1024, 256), (16384, 256, 256)])
def test_small_tile_takes_two_stages_where_three_lose(launches, M, N, K):
    # 64 x 64 tiles against 128 x 128 tiles with two stages: 1.03 and 1.02 times their time with three LDS stages throughout,
    # 0.91 and 0.92 with two where the launch has few k-tiles
    kw = dict(bias=launches.bias, epi=B.EPI_GELU | B.EPI_KEEPGRAD, aux_out=launches.aux)
    small, large = (launches.us(1, M, N, K, impl=impl, **kw) for impl in (105, 107))
    assert small < 0.97 * large


@pytest.mark.parametrize("kc,M,N,K,impl,splits,before", [
    # adding to C, K-contiguous operands
    (1, 2048, 1024, 8192, 106, 6, 1.24), (1, 2048, 1024, 12288, 106, 6, 1.33), (1, 1024, 1024, 16384, 106, 10, 1.24), (1, 3000, 520, 8192, 104, 2, 1.18),
    # ... and K-strided ones
    (0, 64, 1024, 512, 107, 4, 1.23), (0, 256, 256, 512, 107, 4, 1.25), (0, 1000, 136, 512, 107, 4, 1.29),
    # outputs that allow no 16-byte access
    (1, 8192, 257, 256, 105, 0, 1.9)])
def test_accumulating_launches_take_the_fast_tile_and_splits(launches, kc, M, N, K, impl, splits, before):
    # the library's choice of tile and K splits against a forced one that is among the fastest; `before`: what it took relative
    # to that one while the rule priced these launches by the figures of others
    kw = dict(out_f32=True, epi=B.EPI_ACCUM)
    chosen, forced = launches.us(kc, M, N, K, **kw), launches.us(kc, M, N, K, impl=impl, splits=splits, **kw)
    assert chosen < (1 + 0.6 * (before - 1)) * forced
