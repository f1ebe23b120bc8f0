"""Every instance of the GEMM kernel, chosen by its plan: for each (epilogue, tile height, columns per
wavefront, wavefronts, weight caching, split) that hxf_op_gemm can take, small shapes whose plan is
that instance, with K that ends inside a stage, a step and a trip of the pipeline.  Operands are small
integers, so that every order of the sums gives the same fp32 value: fp32 and bf16 results are
compared exactly.  Row-major activations hold NaN past K, and a product of NaN runs first, so that the
workgroups' LDS holds NaN: what a call does not load itself may not reach its result."""
import functools

import pytest

from paper_2505_05286_amd import hxf

from .gpu_util import log, torch

# the instances that launch_wide_cfg and gemm_wide_split name, as (columns per wavefront / 16,
# wavefronts, weights read once): tile heights
UNSPLIT = {(2, 4, 1): {1, 2, 4, 8}, (2, 4, 0): set(range(3, 13)), (4, 4, 1): {1, 2, 4, 6, 8, 10, 12, 14, 16},
           (4, 4, 0): set(range(4, 17)), (4, 8, 0): {9}}
SPLIT = {(2, 4, 1): {1, 2, 4, 8}, (2, 4, 0): set(range(3, 13)), (4, 4, 1): {10, 12, 14, 16},
         (4, 4, 0): set(range(4, 17))}
SPLIT_SWIGLU = {(2, 4, 1): {1, 2, 4, 8}}
KINDS = ["bf16", "resid", "swiglu", "f32", "split", "split_swiglu"]
EPI = {"bf16": hxf.EPI_BF16, "resid": hxf.EPI_RESID, "swiglu": hxf.EPI_SWIGLU, "f32": hxf.EPI_F32,
       "split": hxf.EPI_F32, "split_swiglu": hxf.EPI_SWIGLU}


def instances(kind):
    return {(k, tm) for k, tms in (SPLIT if kind == "split" else SPLIT_SWIGLU if kind == "split_swiglu" else
                                   UNSPLIT).items() for tm in tms}


@functools.lru_cache(None)
def cases(kind):
    """instance -> shapes: the cheapest of each K class."""
    rows = [1, 2, 16, 17, 32, 33, 48, 64, 65, 90, 96, 97, 128] + [16 * r - 3 for r in range(9, 66)] + [177] + [513, 2300]
    cols = [16, 64, 96, 256, 500, 1024, 1376, 1504, 2048, 2560, 3072, 4096, 5120, 5392, 5504, 6144, 7168, 8192, 8224, 10240, 12288,
            14336, 16352, 20480, 22016, 28672, 33000, 40000, 65600]
    depths = ([1024, 2048, 2056, 4096, 8192, 8200, 9728, 11008, 14336, 28672] if kind.startswith("split") else
              [8, 64, 72, 200, 256, 264, 320, 552, 1000])
    best = {}
    for K in depths:
        for N in cols:
            if EPI[kind] == hxf.EPI_SWIGLU and N % 32:
                continue
            for M in rows:
                tm, nw, wv, once, splits, _ = hxf.op_gemm_plan(M, N, K, EPI[kind])
                if (splits > 1) != kind.startswith("split"):
                    continue
                at = best.setdefault(((nw, wv, once), tm), {})
                if K not in at or M * N < at[K][0] * at[K][1]:
                    at[K] = (M, N, K)
    return best


@pytest.mark.parametrize("kind", KINDS)
def test_every_plan_is_an_instance_and_every_instance_is_tested(kind):
    assert set(cases(kind)) == instances(kind)


@pytest.mark.parametrize("kind,narrow,once", [(k, nw, once) for k in KINDS for nw in (2, 4) for once in (0, 1)
                                              if any(i[0][0] == nw and i[0][2] == once for i in instances(k))])
@pytest.mark.gpu
def test_instances(kind, narrow, once):
    t = torch()
    dev = "cuda:0"
    g = t.Generator(device=dev)
    g.manual_seed(5)
    epi, swiglu = EPI[kind], EPI[kind] == hxf.EPI_SWIGLU

    def ints(n, k):
        return t.randint(-4, 5, (n, k), generator=g, device=dev).to(t.bfloat16)

    def packed(w):
        out = t.zeros(hxf.packed_weight_bytes(*w.shape) // 2, dtype=t.bfloat16, device=dev)
        hxf.op_pack_weight(w.data_ptr(), *w.shape, out.data_ptr())
        return out

    nan = t.full((512, 512), float("nan"), dtype=t.bfloat16, device=dev)
    junk = t.empty((512, 24576), dtype=t.float32, device=dev)
    fill = packed(ints(24576, 512))

    def fill_lds():
        """256 rows per workgroup, more of them than CUs: 128 KB of NaN in every LDS."""
        assert hxf.op_gemm_plan(512, 24576, 512, hxf.EPI_F32)[0] >= 14
        hxf.op_gemm(nan.data_ptr(), 512, fill.data_ptr(), 0, junk.data_ptr(), 24576, 512, 24576, 512, hxf.EPI_F32)

    for (key, tm), shapes in sorted(cases(kind).items()):
        if key[0] != narrow or key[2] != once:
            continue
        for M, N, K in shapes.values():
            n_out = N // 2 if swiglu else N
            a, w = ints(M, K), [ints(n_out, K) for _ in range(2 if swiglu else 1)]
            wp = [packed(x) for x in w]
            prod = [a.float() @ x.float().T for x in w]
            wsn = hxf.op_gemm_workspace_bytes(M, N, K)
            ws = t.empty(max(wsn, 256), dtype=t.uint8, device=dev)
            base = t.randint(-9, 10, (M, n_out), generator=g, device=dev).float()
            if swiglu:
                want = (prod[0].double() * t.sigmoid(prod[0].double()) * prod[1].double())
            else:
                want = {hxf.EPI_BF16: prod[0].bfloat16(), hxf.EPI_RESID: base + prod[0], hxf.EPI_F32: prod[0]}[epi]
            for a_packed in ([0, 1] if K % 32 == 0 and not (swiglu and N % 64) else [0]):
                lda = K + 24
                if a_packed:
                    src = packed(a)
                else:
                    src = t.full((M, lda), float("nan"), dtype=t.bfloat16, device=dev)
                    src[:, :K] = a
                if epi == hxf.EPI_RESID:
                    out = base.clone()
                else:
                    out = t.full((M, n_out), float("nan"), device=dev,
                                 dtype=t.float32 if epi == hxf.EPI_F32 else t.bfloat16)
                log(f"{kind} tile {tm} {key} M={M} N={N} K={K} packed={a_packed}")
                fill_lds()
                hxf.op_gemm(src.data_ptr(), lda, wp[0].data_ptr(), wp[1].data_ptr() if swiglu else 0, out.data_ptr(),
                            n_out, M, N, K, epi | (hxf.GEMM_A_PACKED if a_packed else 0), ws.data_ptr(), wsn)
                t.cuda.synchronize()
                if swiglu:
                    # bf16 rounding of the product (2^-9), fp32 sigmoid before it
                    t.testing.assert_close(out.double(), want, rtol=2 ** -8, atol=1e-30)
                else:
                    assert t.equal(out, want)


def _fits(rows, lda, K, tm):
    return ((min(16 * tm, rows) - 1) * lda + K) * 2 < 1 << 31


MI = 1 << 20


@pytest.mark.gpu
@pytest.mark.parametrize("rows,lda,N,K,kind,far", [
    (64, 24 * MI, 64, 72, "f32", False), (65, 24 * MI, 64, 1032, "resid", False), (33, 40 * MI, 128, 1024, "swiglu", False),
    (129, 16 * MI, 22016, 64, "bf16", False), (129, 16 * MI, 22016, 64, "swiglu", False),
    (129, 24 * MI, 22016, 64, "swiglu", False), (150, 32 * MI, 1376, 256, "swiglu", False),
    (17, 72 * MI, 500, 200, "f32", True), (18, 72 * MI, 64, 1032, "bf16", True), (17, 72 * MI, 64, 264, "resid", True),
    (17, 72 * MI, 96, 264, "swiglu", True), (19, 72 * MI, 64, 2056, "swiglu", True)])
def test_row_pitches_beyond_a_tile(rows, lda, N, K, kind, far):
    """A row pitch that puts a planned tile's rows more than 2 GiB apart: a lower tile runs, or, where
    16 rows still span 2 GiB, the kernel with 64-bit addresses; with and without split K."""
    t = torch()
    dev, epi = "cuda:0", EPI[kind]
    assert not _fits(rows, lda, K, hxf.op_gemm_plan(rows, N, K, epi)[0]) and _fits(rows, lda, K, 1) != far
    g = t.Generator(device=dev)
    g.manual_seed(rows + N)
    n_out = N // 2 if kind == "swiglu" else N
    a = t.randint(-4, 5, (rows, K), generator=g, device=dev).to(t.bfloat16)
    w = [t.randint(-4, 5, (n_out, K), generator=g, device=dev).to(t.bfloat16) for _ in range(2)]
    wp = []
    for x in w:
        wp.append(t.zeros(hxf.packed_weight_bytes(n_out, K) // 2, dtype=t.bfloat16, device=dev))
        hxf.op_pack_weight(x.data_ptr(), n_out, K, wp[-1].data_ptr())
    far_apart = t.empty((rows - 1) * lda + K, dtype=t.bfloat16, device=dev)
    far_apart.as_strided((rows, K), (lda, 1)).copy_(a)
    out = t.ones((rows, n_out), dtype=t.float32 if kind in ("f32", "resid") else t.bfloat16, device=dev)
    wsn = hxf.op_gemm_workspace_bytes(rows, N, K)
    ws = t.empty(max(wsn, 256), dtype=t.uint8, device=dev)
    log(f"pitch {rows} x {lda} N={N} K={K} {kind} ws={wsn}")
    hxf.op_gemm(far_apart.data_ptr(), lda, wp[0].data_ptr(), wp[1].data_ptr() if kind == "swiglu" else 0,
                out.data_ptr(), n_out, rows, N, K, epi, ws.data_ptr(), wsn)
    t.cuda.synchronize()
    prod = [a.float() @ x.float().T for x in w]
    if kind == "swiglu":
        d = [x.double() for x in prod]
        t.testing.assert_close(out.double(), d[0] * t.sigmoid(d[0]) * d[1], rtol=2 ** -8, atol=1e-30)
    else:
        assert t.equal(out, {"f32": prod[0], "resid": prod[0] + 1, "bf16": prod[0].bfloat16()}[kind])


@pytest.mark.gpu
@pytest.mark.parametrize("packed", [False, True])
def test_rows_of_more_than_2_gib_of_weights(packed):
    """K so long that the two column tiles of the narrowest form span 2 GiB: split K on 64-bit addresses."""
    t = torch()
    dev, M, N, K = "cuda:0", 2, 16, 34 * MI
    at = t.tensor([0, 7, 63, 1000, 4194303, 4194304, 12345678, K // 2 + 5, K - 9, K - 1], device=dev)
    a = t.zeros((M, K), dtype=t.bfloat16, device=dev)
    w = t.zeros((N, K), dtype=t.bfloat16, device=dev)
    a[:, at] = t.randint(1, 5, (M, len(at)), device=dev).to(t.bfloat16)
    w[:, at] = t.randint(1, 5, (N, len(at)), device=dev).to(t.bfloat16)
    src = a
    wp = t.zeros(hxf.packed_weight_bytes(N, K) // 2, dtype=t.bfloat16, device=dev)
    hxf.op_pack_weight(w.data_ptr(), N, K, wp.data_ptr())
    if packed:
        src = t.zeros(hxf.packed_weight_bytes(M, K) // 2, dtype=t.bfloat16, device=dev)
        hxf.op_pack_weight(a.data_ptr(), M, K, src.data_ptr())
    out = t.zeros((M, N), dtype=t.float32, device=dev)
    ws = t.empty(hxf.op_gemm_workspace_bytes(M, N, K), dtype=t.uint8, device=dev)
    log(f"long K, packed={packed}, plan {hxf.op_gemm_plan(M, N, K, hxf.EPI_F32)}")
    hxf.op_gemm(src.data_ptr(), K, wp.data_ptr(), 0, out.data_ptr(), N, M, N, K,
                hxf.EPI_F32 | (hxf.GEMM_A_PACKED if packed else 0), ws.data_ptr(), ws.numel())
    t.cuda.synchronize()
    assert t.equal(out, a[:, at].float() @ w[:, at].float().T)
