"""Parity of the HIP path (through the C ABI) against the CPU oracle, element by
element on the same seeded inputs.  Integer work (packing, quantized
activations, int32 accumulators) must match bit for bit; floating-point outputs
must satisfy the floored relative error bound 2e-3 (fp32 accumulation, binary16
output)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2505_00232_amd import binding, synth

pytestmark = pytest.mark.gpu
TOL = 2e-3
DEV = "cuda"


def _layer(wq, s, fmt, max_m=8, mode=None):
    return binding.QuantLinear(wq, s, fmt, compute_mode=mode, max_m=max_m)


def _group(fmt):
    return 32 if fmt == "w4g32" else 0


def _E(y, ref) -> float:
    """The acceptance metric (floored relative error), and beside it the plain maximum relative
    error over the entries at or above their row's floor, which the same bound must hold for."""
    e = oracle.floored_rel_error(y, ref)
    p = oracle.plain_rel_error_above_floor(y, ref)
    assert p <= e * (1 + 1e-12) + 1e-300, (p, e)
    return max(e, p)


def _forward(layer, x):
    xd = torch.from_numpy(x).to(DEV)
    y = layer.forward(xd)
    torch.cuda.synchronize()
    return y.cpu().numpy()


# ------------------------------------------------------------------ A1 pack / unpack
@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(1, 32), (17, 96), (64, 256), (300, 512), (1000, 2304)])
def test_pack_unpack_round_trip_bit_exact(fmt, N, K):
    print(f"pack/unpack {fmt} N={N} K={K}", flush=True)
    rng = np.random.default_rng(N * 7919 + K)
    if fmt == "w8c":
        wq = rng.integers(-128, 128, size=(N, K), dtype=np.int8)
        wq.flat[: min(256, wq.size)] = np.arange(-128, 128, dtype=np.int16).astype(np.int8)[: min(256, wq.size)]
        s = rng.integers(0, 2**32, size=N, dtype=np.uint32).view(np.float32)  # any bit pattern
    else:
        wq = rng.integers(-8, 8, size=(N, K), dtype=np.int8)
        wq.flat[:16] = np.arange(-8, 8, dtype=np.int8)
        if fmt == "w4c":
            s = rng.integers(0, 2**32, size=N, dtype=np.uint32).view(np.float32)
        else:
            s = rng.integers(0, 2**16, size=(N, K // 32), dtype=np.uint16).view(np.float16)
    per_channel = fmt != "w4g32"
    layer = _layer(wq, s, fmt)
    wq_back = torch.full((N, K), 99, dtype=torch.int8, device=DEV)
    s_back = torch.zeros(s.shape, dtype=torch.float32 if per_channel else torch.float16, device=DEV)
    binding.qfc_unpack_weights(layer.handle, wq_back, s_back)
    torch.cuda.synchronize()
    assert np.array_equal(wq_back.cpu().numpy(), wq)
    sb = s_back.cpu().numpy()
    assert np.array_equal(sb.view(np.uint32 if per_channel else np.uint16),
                          s.view(np.uint32 if per_channel else np.uint16))
    layer.close()


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(17, 96), (300, 512), (1000, 2304), (129, 14336)])
def test_embedding_lookup_bit_exact(fmt, N, K):
    """Rows of the packed table as binary16: the same bits as the oracle (fp32 product, one rounding to
    binary16), ids out of range give zeros, the rows of y past M stay untouched."""
    print(f"embedding {fmt} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(2500, N, K, fc)
    layer = _layer(wq, s, fmt)
    rng = np.random.default_rng(N + K)
    ids = np.concatenate([[0, N - 1, -3, N], rng.integers(0, N, size=9)]).astype(np.int32)
    M = len(ids)
    y = torch.full((M + 1, K), 3.0, dtype=torch.float16, device=DEV)
    binding.qfc_embedding(layer.handle, torch.from_numpy(ids).to(DEV), y[:M])  # (a view of the first M rows)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    ref = oracle.embedding(ids, wq, s, _group(fmt))
    assert np.array_equal(got[:M].view(np.uint16), ref.view(np.uint16))
    assert np.all(got[M] == np.float16(3.0))
    layer.close()


# ------------------------------------------------------------------ A2 decode
# (48, 6144): 12 units of the int8 format, 6 of the int4 formats, i.e. the plans with more than 8
# wavefronts (int8) and with full units at a medium K (int4); (96, 14336): 14 / 28 units
DECODE_SHAPES = [(1, 32), (17, 96), (130, 256), (1000, 2304), (96, 14336), (1024, 512), (48, 6144)]


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", DECODE_SHAPES)
def test_decode_matches_oracle(fmt, N, K):
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(2000, N, K, fc)
    wq.flat[0] = -128 if fmt == "w8c" else -8
    layer = _layer(wq, s, fmt)
    for M in range(1, 9):
        print(f"decode {fmt} N={N} K={K} M={M}", flush=True)
        x = synth.activations(2000, N, K + M, M, K)
        y = _forward(layer, x)
        ref = oracle.fc_weight_only(x, wq, s, _group(fmt))
        err = _E(y, ref)
        assert err <= TOL, (M, err)
        y2 = _forward(layer, x)
        assert np.array_equal(y.view(np.uint16), y2.view(np.uint16))  # deterministic
    layer.close()


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
def test_decode_config1_and_structure_cases(fmt):
    print(f"decode structure cases {fmt}", flush=True)
    # identity weights with unit scales return x bit for bit (one non-zero term per output)
    K = 512
    eye = np.eye(K, dtype=np.int8)
    ones = np.ones(K, np.float32) if fmt != "w4g32" else np.ones((K, K // 32), np.float16)
    layer = _layer(eye, ones, fmt)
    x = synth.activations(2001, 0, 0, 4, K)
    y = _forward(layer, x)
    assert np.array_equal(y.view(np.uint16), x.view(np.uint16))
    layer.close()
    # one-hot rows with power-of-two scales: y[m,n] = s_n q_n x[m, perm(n)] exactly
    rng = np.random.default_rng(11)
    N, K = 700, 1024
    perm = rng.integers(0, K, size=N)
    q = rng.integers(1, 8, size=N) * rng.choice([-1, 1], size=N)
    wq = np.zeros((N, K), np.int8)
    wq[np.arange(N), perm] = q
    if fmt != "w4g32":
        s = (2.0 ** rng.integers(-6, 3, size=N)).astype(np.float32)
        sn = s.astype(np.float64)
    else:
        s = (2.0 ** rng.integers(-6, 3, size=(N, K // 32))).astype(np.float16)
        sn = s.astype(np.float64)[np.arange(N), perm // 32]
    layer = _layer(wq, s, fmt)
    x = synth.activations(2002, 0, 0, 3, K)
    y = _forward(layer, x)
    want = (x.astype(np.float64)[:, perm] * (sn * q)[None, :]).astype(np.float16)
    assert np.array_equal(y.view(np.uint16), want.view(np.uint16))
    assert np.array_equal(oracle.fc_weight_only(x, wq, s, _group(fmt)).astype(np.float16).view(np.uint16),
                          want.view(np.uint16))
    layer.close()


def test_decode_config1():
    print("config 1", flush=True)
    fc = synth.CFG1_FC
    wq, s = synth.weights(1001, 0, 0, fc)
    x = synth.activations(1001, 0, 0, 1, fc.K)
    layer = _layer(wq, s, fc.fmt)
    y = _forward(layer, x)
    assert _E(y, oracle.fc_weight_only(x, wq, s)) <= TOL
    layer.close()


def test_decode_config2_gemma_layer_full():
    for i, fc in enumerate(synth.GEMMA_FCS_W4):
        print(f"config 2 {fc.name} {fc.K}->{fc.N}", flush=True)
        wq, s = synth.weights(1002, 0, i, fc)
        x = synth.activations(1002, 0, i, 1, fc.K)
        layer = _layer(wq, s, fc.fmt)
        y = _forward(layer, x)
        assert _E(y, oracle.fc_weight_only(x, wq, s, 32)) <= TOL
        layer.close()


@pytest.mark.parametrize("M", [1, 4])
def test_decode_config3_llama_shapes_sampled(M):
    """Full-size Llama-3.1-8B FCs in the launch configuration the benchmark
    uses; the oracle evaluates a random sample of output channels."""
    rng = np.random.default_rng(3)
    for i, fc in enumerate(synth.LLAMA_FCS_W4 + (synth.LLAMA_LM_HEAD,)):
        print(f"config 3 {fc.name} {fc.K}->{fc.N} M={M}", flush=True)
        wq, s = synth.weights(1003, 0, i, fc)
        x = synth.activations(1003, 0, i, M, fc.K)
        layer = _layer(wq, s, fc.fmt)
        y = _forward(layer, x)
        rows = np.sort(rng.choice(fc.N, size=1536, replace=False))
        rows[:2] = (0, 1)
        rows[-2:] = (fc.N - 2, fc.N - 1)
        ref = oracle.fc_weight_only(x, wq[rows], s[rows], _group(fc.fmt))
        assert _E(y[:, rows], ref) <= TOL
        assert np.all(np.isfinite(y.astype(np.float32)))
        layer.close()
        del wq, s


# ------------------------------------------------------------------ A3 activation quantization
@pytest.mark.parametrize("M,K", [(1, 32), (5, 96), (64, 14336), (1024, 4096)])
def test_activation_quantization_bit_exact(M, K):
    print(f"act quant M={M} K={K}", flush=True)
    x = synth.activations(3000, M, K, M, K)
    if M >= 5:
        x[1] = 0
        x[2] = (x[2].astype(np.float32) * 2.0**-12).astype(np.float16)
        x[3, 0] = np.float16(65504.0)
        x[4, :] = np.float16(-3.0)
    xd = torch.from_numpy(x).to(DEV)
    xq = torch.empty((M, K), dtype=torch.int8, device=DEV)
    sx = torch.empty((M,), dtype=torch.float32, device=DEV)
    binding.qfc_quantize_activations(xd, xq, sx)
    torch.cuda.synchronize()
    xq_ref, sx_ref = oracle.quantize_activations(x)
    assert np.array_equal(sx.cpu().numpy().view(np.uint32), sx_ref.view(np.uint32))
    assert np.array_equal(xq.cpu().numpy(), xq_ref)


# ------------------------------------------------------------------ A4 / A5 int8 prefill
@pytest.mark.parametrize("M,N,K", [(9, 1, 32), (100, 130, 96), (200, 300, 512), (256, 1000, 2304), (130, 64, 14336)])
def test_int8_prefill_matches_oracle(M, N, K):
    print(f"int8 prefill M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, "w8c")
    wq, sw = synth.weights(4000, M, N, fc)
    wq.flat[0] = -128
    x = synth.activations(4000, M, N, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    xq_d = torch.from_numpy(xq_ref).to(DEV)
    acc = torch.empty((M, N), dtype=torch.int32, device=DEV)
    binding.qfc_forward_acc_i32(layer.handle, xq_d, acc)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref)
    y = torch.empty((M, N), dtype=torch.float16, device=DEV)
    binding.qfc_forward_q8(layer.handle, xq_d, torch.from_numpy(sx_ref).to(DEV), y)
    torch.cuda.synchronize()
    assert _E(y.cpu().numpy(), y_ref) <= TOL
    y2 = _forward(layer, x)  # quantization kernel + product + epilogue in one call
    assert _E(y2, y_ref) <= TOL
    layer.close()


@pytest.mark.parametrize("M,N,K", [(512, 4096, 4096), (1024, 6144, 4096)])
def test_int8_prefill_whole_output_against_oracle(M, N, K):
    """Every element of a mid-size layer and of the QKV layer of the Llama-3.1-8B prefill workload
    (all workgroups of a real launch, not a sample): quantized activations and int32 accumulators
    bit for bit, outputs within the tolerance."""
    print(f"int8 prefill whole output vs oracle M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, "w8c")
    wq, sw = synth.weights(4100, M, N, fc)
    x = synth.activations(4100, M, N, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    acc = torch.empty((M, N), dtype=torch.int32, device=DEV)
    binding.qfc_forward_acc_i32(layer.handle, torch.from_numpy(xq_ref).to(DEV), acc)
    y = _forward(layer, x)
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref)
    assert _E(y, y_ref) <= TOL
    layer.close()


# The paper's own "8/4/4" scheme in the prefill stage: int8 activations x int4 per-channel weights
@pytest.mark.parametrize("M,N,K", [(9, 1, 32), (100, 130, 96), (200, 300, 512), (256, 1000, 2304), (130, 64, 14336),
                                   (513, 264, 128), (300, 4096, 1152), (77, 300, 256)])
def test_int8_prefill_int4_weights_matches_oracle(M, N, K):
    print(f"int8 x int4 prefill M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, "w4c")
    wq, sw = synth.weights(4500, M, N, fc)
    wq.flat[0], wq.flat[1] = -8, 7
    x = synth.activations(4500, M, N, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    layer = _layer(wq, sw, "w4c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    xq_d = torch.from_numpy(xq_ref).to(DEV)
    acc = torch.empty((M, N), dtype=torch.int32, device=DEV)
    for rep in range(2):
        acc.fill_(-1)
        binding.qfc_forward_acc_i32(layer.handle, xq_d, acc)
        torch.cuda.synchronize()
        assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), rep
    y = torch.empty((M, N), dtype=torch.float16, device=DEV)
    binding.qfc_forward_q8(layer.handle, xq_d, torch.from_numpy(sx_ref).to(DEV), y)
    torch.cuda.synchronize()
    assert _E(y.cpu().numpy(), y_ref) <= TOL
    y2 = _forward(layer, x)  # quantization kernel (codes in the order of the packed weights) + product + epilogue
    assert _E(y2, y_ref) <= TOL
    # the two routes to the activations' codes give the same bits
    assert np.array_equal(y2.view(np.uint16), y.cpu().numpy().view(np.uint16))
    # decode through the same handle keeps binary16 activations
    y1 = _forward(layer, x[:3])
    assert _E(y1, oracle.fc_weight_only(x[:3], wq, sw, 0)) <= TOL
    # fused input gate and residual, as for 8-bit weights
    gate = synth.activations(4501, M, N, M, K)
    res = synth.activations(4502, M, N, M, N)
    yf = _fused(layer, x, gate, binding.QFC_ACT_SILU, res)
    assert _E(yf, _fused_ref(x, wq, sw, "w4c", gate, oracle.SILU, res, int8_act=True)) <= TOL
    layer.close()


def test_int8_prefill_int4_weights_llama_ffn_shapes_sampled():
    """gate+up and down projections of the Llama-3.1-8B layer at M = 1024 with int4 per-channel weights
    (the "8/4/4" FFN): accumulators of sampled rows and channels bit for bit, outputs within the tolerance."""
    rng = np.random.default_rng(45)
    M = 1024
    for i, fc in enumerate(synth.LLAMA_FCS_W4C[2:], start=2):
        print(f"int8 x int4 prefill {fc.name} {fc.K}->{fc.N}", flush=True)
        wq, sw = synth.weights(1104, 0, i, fc)
        x = synth.activations(1104, 0, i, M, fc.K)
        layer = _layer(wq, sw, "w4c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
        xq_ref, sx_ref = oracle.quantize_activations(x)
        acc = torch.empty((M, fc.N), dtype=torch.int32, device=DEV)
        binding.qfc_forward_acc_i32(layer.handle, torch.from_numpy(xq_ref).to(DEV), acc)
        y = _forward(layer, x)
        rows = np.sort(rng.choice(M, size=48, replace=False))
        cols = np.sort(rng.choice(fc.N, size=384, replace=False))
        rows[0], rows[-1], cols[0], cols[-1] = 0, M - 1, 0, fc.N - 1
        acc_ref = oracle.int_contract(xq_ref[rows], wq[cols])
        assert np.array_equal(acc.cpu().numpy()[np.ix_(rows, cols)].astype(np.int64), acc_ref)
        y_ref = oracle.rescale(acc_ref, sx_ref[rows], sw[cols])
        assert _E(y[np.ix_(rows, cols)], y_ref) <= TOL
        layer.close()


@pytest.mark.parametrize("N,K,M,residual", [(65564, 1024, 9, False), (65535, 992, 17, True), (40961, 4096, 32, False), (40964, 4064, 16, True), (32768, 8192, 25, False)])
def test_int8_few_rows_of_many_channels(N, K, M, residual):
    """Layers whose workgroups stay and walk over row tiles (odd counts of them, ragged channels, k and rows): the sums are whole numbers,
    so the outputs are those of the kernel with one workgroup per few row tiles, bit for bit, and right where the oracle looks."""
    print(f"int8 few rows of many channels N={N} K={K} M={M} residual={residual}", flush=True)
    gen = torch.Generator().manual_seed(N + K + M)
    wq = torch.randint(-127, 128, (N, K), generator=gen, dtype=torch.int8)
    sw = torch.rand(N, generator=gen) * 1e-3 + 1e-4
    x = torch.randn((M, K), generator=gen).half()
    res = torch.randn((M, N), generator=gen).half() if residual else None
    layer = binding.QuantLinear(wq.to(DEV), sw.to(DEV), "w8c", compute_mode=1, max_m=M)
    xd, rd = x.to(DEV), res.to(DEV) if residual else None
    outs = []
    try:
        for blocks in (0, 1):  # 1: the other kernel
            binding.qfc_tune(11, blocks)
            y = torch.full((M, N), 9.0, dtype=torch.float16, device=DEV)
            if residual:
                binding.qfc_forward_fused(layer.handle, xd, y, residual=rd)
            else:
                binding.qfc_forward(layer.handle, xd, y)
            outs.append(y)
        torch.cuda.synchronize()
    finally:
        binding.qfc_tune(11, 0)
        layer.close()
    assert torch.equal(outs[0], outs[1])
    if not residual:
        cols = np.unique(np.concatenate([np.arange(40), np.arange(N - 70, N), np.random.default_rng(N).integers(0, N, 200)]))
        y_ref = oracle.fc_int8_act(x.numpy(), wq.numpy()[cols], sw.numpy()[cols])[3]
        assert _E(outs[0].cpu().numpy()[:, cols], y_ref) <= TOL


@pytest.mark.parametrize("variant", [4, 10, 12])
def test_int8_prefill_other_tile_shapes_bit_exact(variant):
    """The kernels of the int8 product (both operands staged; weights straight into registers with 128 and 64 token rows per
    workgroup), forced on a ragged shape."""
    print(f"int8 prefill tile variant {variant}", flush=True)
    M, N, K = 300, 520, 1152
    fc = synth.FC("t", K, N, "w8c")
    wq, sw = synth.weights(4100, M, N, fc)
    x = synth.activations(4100, M, N, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    layer = _layer(wq, sw, "w8c", max_m=M)
    binding.qfc_tune(2, variant)
    try:
        # (three times: a launch that is not the first of its kernel in the process runs with warm
        # caches and different timing, which once exposed a register reused under an unfinished load)
        for rep in range(3):
            acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
            binding.qfc_forward_acc_i32(layer.handle, torch.from_numpy(xq_ref).to(DEV), acc)
            y = _forward(layer, x)
            assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), rep
            assert _E(y, y_ref) <= TOL, rep
    finally:
        binding.qfc_tune(2, 0)
    layer.close()


@pytest.mark.parametrize("variant", [20, 21, 23])
def test_int8_prefill_int4_weights_tile_shapes_bit_exact(variant):
    """The kernels of the int8 x int4 product (both operands staged; weights straight into registers
    with 128 and 64 token rows per workgroup), forced on a ragged shape."""
    print(f"int8 x int4 prefill tile variant {variant}", flush=True)
    M, N, K = 300, 520, 1024
    fc = synth.FC("t", K, N, "w4c")
    wq, sw = synth.weights(4600, M, N, fc)
    x = synth.activations(4600, M, N, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    layer = _layer(wq, sw, "w4c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    binding.qfc_tune(2, variant)
    try:
        for rep in range(3):
            acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
            binding.qfc_forward_acc_i32(layer.handle, torch.from_numpy(xq_ref).to(DEV), acc)
            y = _forward(layer, x)
            assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), rep
            assert _E(y, y_ref) <= TOL, rep
    finally:
        binding.qfc_tune(2, 0)
    layer.close()


@pytest.mark.parametrize("fmt,variant,M,N,K", [
    # two parts of K: the fewest stages, one pair of stages more in the first part, many; ragged channels and token rows, rows stored value by value,
    # one token tile and more of them than share the prefetch
    ("w8c", 13, 131, 600, 512), ("w8c", 13, 300, 523, 768), ("w8c", 13, 65, 129, 6144), ("w8c", 13, 2200, 136, 1280), ("w8c", 14, 131, 600, 512),
    ("w8c", 14, 64, 257, 768), ("w8c", 14, 300, 520, 2304), ("w8c", 14, 1100, 136, 1280), ("w8c", 10, 1930, 257, 768), ("w8c", 10, 1030, 777, 4352),
    ("w4c", 24, 131, 600, 512), ("w4c", 24, 64, 257, 768), ("w4c", 24, 300, 523, 2304), ("w4c", 24, 65, 520, 5632),
    # four parts: one, two and three of them with a pair of stages more
    ("w4c", 25, 131, 600, 1024), ("w4c", 25, 300, 129, 1280), ("w4c", 25, 65, 523, 1536), ("w4c", 25, 64, 129, 1792), ("w4c", 25, 300, 520, 5120)])
def test_int8_tiles_parts_of_k_bit_exact(fmt, variant, M, N, K):
    """The tiles whose groups of wavefronts each take a part of K: sums handed over through LDS, bit for bit, three times (warm
    caches); with a residual."""
    print(f"int8 tiles, K in parts, {fmt} variant {variant} M={M} N={N} K={K}", flush=True)
    wq, sw = synth.weights(4670, M, K, synth.FC("t", K, N, fmt))
    x = synth.activations(4670, M, K, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    res = synth.activations(4671, M, N, M, N)
    layer = _layer(wq, sw, fmt, max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    binding.qfc_tune(2, variant)
    try:
        for rep in range(3):
            acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
            binding.qfc_forward_acc_i32(layer.handle, torch.from_numpy(xq_ref).to(DEV), acc)
            y = _forward(layer, x)
            assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), rep
            assert _E(y, y_ref) <= TOL, rep
        out = torch.empty((M, N), dtype=torch.float16, device=DEV)
        binding.qfc_forward_fused(layer.handle, torch.from_numpy(x).to(DEV), out, residual=torch.from_numpy(res).to(DEV))
        assert _E(out.cpu().numpy(), y_ref + res.astype(np.float64)) <= TOL
    finally:
        binding.qfc_tune(2, 0)
    layer.close()


@pytest.mark.parametrize("fmt,variant,M,N,K", [
    # one channel tile and ragged ones, one token tile and ragged ones (whole and half groups without a row to store), parts of K of unequal length; and the forms
    # with K in one part
    *[("w8c", v, *s) for v in (13, 14) for s in ((131, 608, 512), (64, 32, 768), (300, 160, 1280), (33, 544, 2304))],
    *[("w4c", 24, *s) for s in ((131, 608, 512), (64, 32, 768), (300, 160, 1280), (33, 544, 2304))],
    *[("w4c", 25, *s) for s in ((131, 608, 1024), (64, 32, 1280), (300, 160, 1536), (33, 544, 1792), (300, 544, 2304))],
    ("w8c", 10, 131, 608, 512), ("w8c", 12, 131, 608, 512), ("w4c", 21, 131, 608, 512), ("w4c", 23, 131, 608, 512),
    # large enough for the choice by size to go there: forms 14, 13, 24, 25
    ("w8c", 0, 700, 2048, 2304), ("w8c", 0, 1500, 2048, 4096), ("w4c", 0, 300, 4096, 4096), ("w4c", 0, 814, 2304, 9216)])
def test_int8_tiles_gated_output(fmt, variant, M, N, K):
    """act(gate) * up in the store phase of every form of the direct-weights int8 tiles, above all those whose groups of wavefronts hand their sums over
    and store half of the token rows each; a row past the last stays as it was."""
    print(f"int8 tiles, gated output, {fmt} variant {variant} M={M} N={N} K={K}", flush=True)
    wq, sw = synth.weights(4680, M, K, synth.FC("t", K, N, fmt))
    x = (synth.activations(4680, M, K, M, K) * np.float16(0.125)).astype(np.float16)
    layer = binding.QuantLinear(wq, sw, fmt, compute_mode=binding.QFC_COMPUTE_INT8_ACT, max_m=M, gated_pairs=True)
    guard = torch.full((M + 1, N // 2), 77.0, dtype=torch.float16, device=DEV)
    xd = torch.from_numpy(x).to(DEV)
    rows = np.arange(M) if M * N * K < 1 << 29 else np.unique(np.concatenate([[0, M - 1], np.random.default_rng(M).integers(0, M, 62)]))
    ref = oracle.gated_output(oracle.fc_int8_act(x[rows], wq, sw)[3], oracle.SILU)
    binding.qfc_tune(2, variant)
    try:
        for rep in range(2):
            guard[:M] = 55.0
            binding.qfc_forward_fused(layer.handle, xd, guard[:M], activation=binding.QFC_ACT_SILU, gated_output=True)
            torch.cuda.synchronize()
            assert _E(guard[:M].cpu().numpy()[rows], ref) <= TOL, rep
            assert bool((guard[M] == 77.0).all())
    finally:
        binding.qfc_tune(2, 0)
    layer.close()


@pytest.mark.parametrize("fmt,K", [("w4c", 256), ("w4c", 512), ("w4c", 768), ("w4c", 2304), ("w4c", 2560), ("w8c", 256), ("w8c", 512), ("w8c", 2400), ("w8c", 6144), ("w8c", 6400), ("w8c", 7168), ("w8c", 7392)])
def test_int8_tiles_of_64_tokens_any_even_number_of_stages(fmt, K):
    """The 64-token tiles, which hold the weights of four stages of 128 k (int8 codes: of two): whole passes of four, two
    stages more, only two, and K that ends inside a stage; three channel tiles and three token tiles, the last ones ragged; bit for bit,
    and the same again with warm caches."""
    M, N = 131, 600
    print(f"int8 tiles of 64 tokens {fmt} K={K}", flush=True)
    wq, sw = synth.weights(4650, M, K, synth.FC("t", K, N, fmt))
    x = synth.activations(4650, M, K, M, K)
    xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
    layer = _layer(wq, sw, fmt, max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    xq_d = torch.from_numpy(xq_ref).to(DEV)
    binding.qfc_tune(2, 12 if fmt == "w8c" else 23)
    try:
        for rep in range(3):
            acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
            binding.qfc_forward_acc_i32(layer.handle, xq_d, acc)
            y = _forward(layer, x)
            assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), rep
            assert _E(y, y_ref) <= TOL, rep
    finally:
        binding.qfc_tune(2, 0)
    layer.close()


def test_int8_prefill_config4_shapes_sampled():
    """Llama layer at M = 1024, int8 per-channel weights: accumulators of a
    sample of (token, channel) pairs against the exact integer contraction."""
    rng = np.random.default_rng(4)
    M = 1024
    for i, fc in enumerate(synth.LLAMA_FCS_W8):
        print(f"config 4 {fc.name} {fc.K}->{fc.N}", flush=True)
        wq, sw = synth.weights(1004, 0, i, fc)
        x = synth.activations(1004, 0, i, M, fc.K)
        layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
        xd = torch.from_numpy(x).to(DEV)
        xq = torch.empty((M, fc.K), dtype=torch.int8, device=DEV)
        sx = torch.empty((M,), dtype=torch.float32, device=DEV)
        binding.qfc_quantize_activations(xd, xq, sx)
        acc = torch.empty((M, fc.N), dtype=torch.int32, device=DEV)
        binding.qfc_forward_acc_i32(layer.handle, xq, acc)
        y = layer.forward(xd)
        torch.cuda.synchronize()
        xq_ref, sx_ref = oracle.quantize_activations(x)
        assert np.array_equal(xq.cpu().numpy(), xq_ref)
        assert np.array_equal(sx.cpu().numpy().view(np.uint32), sx_ref.view(np.uint32))
        rows = np.sort(rng.choice(M, size=48, replace=False))
        cols = np.sort(rng.choice(fc.N, size=384, replace=False))
        rows[0], rows[-1], cols[0], cols[-1] = 0, M - 1, 0, fc.N - 1
        acc_ref = oracle.int_contract(xq_ref[rows], wq[cols])
        got = acc.cpu().numpy()[np.ix_(rows, cols)].astype(np.int64)
        assert np.array_equal(got, acc_ref)
        y_ref = oracle.rescale(acc_ref, sx_ref[rows], sw[cols])
        assert _E(y.cpu().numpy()[np.ix_(rows, cols)], y_ref) <= TOL
        layer.close()
        del wq


def test_int8_prefill_config5_lm_head_sampled():
    """Gemma2-2B LM head (2304 -> 256000, int8 per-channel) at M = 2048: quantized
    activations bit for bit, sampled accumulators against the exact contraction,
    sampled outputs within tolerance."""
    print("config 5 lm head", flush=True)
    rng = np.random.default_rng(55)
    M, fc = 2048, synth.GEMMA_LM_HEAD
    wq, sw = synth.weights(1005, 0, 4, fc)
    x = synth.activations(1005, 0, 4, M, fc.K)
    layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    xd = torch.from_numpy(x).to(DEV)
    xq = torch.empty((M, fc.K), dtype=torch.int8, device=DEV)
    sx = torch.empty((M,), dtype=torch.float32, device=DEV)
    binding.qfc_quantize_activations(xd, xq, sx)
    acc = torch.empty((M, fc.N), dtype=torch.int32, device=DEV)
    binding.qfc_forward_acc_i32(layer.handle, xq, acc)
    y = layer.forward(xd)
    torch.cuda.synchronize()
    xq_ref, sx_ref = oracle.quantize_activations(x)
    assert np.array_equal(xq.cpu().numpy(), xq_ref)
    assert np.array_equal(sx.cpu().numpy().view(np.uint32), sx_ref.view(np.uint32))
    rows = np.sort(rng.choice(M, size=32, replace=False))
    cols = np.sort(rng.choice(fc.N, size=512, replace=False))
    rows[0], rows[-1], cols[0], cols[-1] = 0, M - 1, 0, fc.N - 1
    ri, ci = torch.from_numpy(rows).to(DEV), torch.from_numpy(cols).to(DEV)
    acc_ref = oracle.int_contract(xq_ref[rows], wq[cols])
    assert np.array_equal(acc[ri][:, ci].cpu().numpy().astype(np.int64), acc_ref)
    y_ref = oracle.rescale(acc_ref, sx_ref[rows], sw[cols])
    assert _E(y[ri][:, ci].cpu().numpy(), y_ref) <= TOL
    layer.close()


@pytest.mark.parametrize("M,N,K", [(2048, 28672, 4096), (1024, 4096, 14336)])
def test_int8_prefill_whole_output_at_many_workgroups_per_compute_unit(M, N, K):
    """Launches of several rounds of workgroups per compute unit (the store phase of a workgroup
    reuses the LDS ring that its own last copies still target).  Sampled accumulators against the
    exact contraction; then, over the whole output: the two kernel families (weights straight into
    registers / both operands through LDS) give the same accumulators, and y is the scaled
    accumulator bit for bit (two fp32 multiplications and one rounding to binary16, in that
    order; no oracle value is involved in that last comparison, only the definition)."""
    print(f"int8 prefill whole output M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M + N)
    fc = synth.FC("t", K, N, "w8c")
    wq, sw = synth.weights(4200, M, N, fc)
    x = synth.activations(4200, M, N, M, K)
    layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    xd = torch.from_numpy(x).to(DEV)
    xq = torch.empty((M, K), dtype=torch.int8, device=DEV)
    sx = torch.empty((M,), dtype=torch.float32, device=DEV)
    binding.qfc_quantize_activations(xd, xq, sx)
    acc = torch.empty((M, N), dtype=torch.int32, device=DEV)
    acc_lds = torch.empty((M, N), dtype=torch.int32, device=DEV)
    y = torch.empty((M, N), dtype=torch.float16, device=DEV)
    for rep in range(3):  # (the failure this guards against depended on timing)
        acc.fill_(-1)
        y.fill_(-1.0)
        binding.qfc_forward_acc_i32(layer.handle, xq, acc)
        binding.qfc_forward_q8(layer.handle, xq, sx, y)
        binding.qfc_tune(2, 4)
        try:
            binding.qfc_forward_acc_i32(layer.handle, xq, acc_lds)
        finally:
            binding.qfc_tune(2, 0)
        torch.cuda.synchronize()
        if rep == 0:
            xq_ref, _ = oracle.quantize_activations(x)
            rows = np.sort(rng.choice(M, size=8, replace=False))
            cols = np.sort(rng.choice(N, size=512, replace=False))
            acc_ref = oracle.int_contract(xq_ref[rows], wq[cols])
            ri, ci = torch.from_numpy(rows).to(DEV), torch.from_numpy(cols).to(DEV)
            assert np.array_equal(acc[ri][:, ci].cpu().numpy().astype(np.int64), acc_ref)
        assert torch.equal(acc, acc_lds)
        expected = ((acc.float() * sx[:, None]) * torch.from_numpy(sw).to(DEV)[None, :]).half()
        assert torch.equal(y, expected)
    layer.close()


# ------------------------------------------------------------------ A6 fp16 MFMA prefill with in-LDS dequantization
@pytest.mark.parametrize("fmt", ["w4g32", "w4c"])
@pytest.mark.parametrize("M,N,K", [(9, 1, 32), (100, 130, 96), (200, 300, 512), (130, 1000, 2304),
                                   (300, 264, 128), (129, 520, 1152), (16, 256, 2176)])
def test_fp16_prefill_matches_oracle(fmt, M, N, K):
    print(f"fp16 prefill {fmt} M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(5000, M, N, fc)
    wq.flat[0] = -8
    x = synth.activations(5000, M, N, M, K)
    layer = _layer(wq, s, fmt, max_m=M)
    y = _forward(layer, x)
    ref = oracle.fc_weight_only(x, wq, s, _group(fmt))
    assert _E(y, ref) <= TOL
    layer.close()


@pytest.mark.parametrize("fmt,M,N,K", [("w4g32", 512, 4096, 4096), ("w4c", 512, 4096, 4096), ("w4g32", 2048, 4096, 2304)])
def test_fp16_prefill_whole_output_against_oracle(fmt, M, N, K):
    """Every element of a mid-size layer, and of the QKV layer of the Gemma2-2B prefill workload at
    its full M = 2048, against the oracle (not a sample)."""
    print(f"fp16 prefill whole output vs oracle {fmt} M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(5100, M, N, fc)
    x = synth.activations(5100, M, N, M, K)
    layer = _layer(wq, s, fmt, max_m=M)
    y = _forward(layer, x)
    assert _E(y, oracle.fc_weight_only(x, wq, s, _group(fmt))) <= TOL
    layer.close()


@pytest.mark.parametrize("M,N,K", [(9, 1, 32), (100, 130, 96), (200, 300, 512), (130, 1000, 2304), (64, 264, 14336)])
def test_fp16_prefill_int8_weights_matches_oracle(M, N, K):
    """Per-channel int8 weights with binary16 activations at M > 8 (the "q8" scheme with FP16
    activations): the weight-only definition, as for the int4 formats; residual merged as there."""
    print(f"fp16 prefill w8c M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, "w8c")
    wq, s = synth.weights(5200, M, N, fc)
    wq.flat[0], wq.flat[1] = -128, 127
    x = synth.activations(5200, M, N, M, K)
    layer = _layer(wq, s, "w8c", max_m=M, mode=binding.QFC_COMPUTE_FP16_DEQUANT)
    ref = oracle.fc_weight_only(x, wq, s, 0)
    assert _E(_forward(layer, x), ref) <= TOL
    res = synth.activations(5201, M, N, M, N)
    assert _E(_fused(layer, x, None, 0, res), oracle.add_residual(ref, res)) <= TOL
    # decode through the same handle
    assert _E(_forward(layer, x[:5]), ref[:5]) <= TOL
    layer.close()


def test_fp16_prefill_config5_shapes_sampled():
    rng = np.random.default_rng(5)
    M = 2048
    for i, fc in enumerate(synth.GEMMA_FCS_W4):
        print(f"config 5 {fc.name} {fc.K}->{fc.N}", flush=True)
        wq, s = synth.weights(1005, 0, i, fc)
        x = synth.activations(1005, 0, i, M, fc.K)
        layer = _layer(wq, s, "w4g32", max_m=M)
        y = _forward(layer, x)
        rows = np.sort(rng.choice(M, size=64, replace=False))
        cols = np.sort(rng.choice(fc.N, size=512, replace=False))
        rows[0], rows[-1], cols[0], cols[-1] = 0, M - 1, 0, fc.N - 1
        ref = oracle.fc_weight_only(x[rows], wq[cols], s[cols], 32)
        assert _E(y[np.ix_(rows, cols)], ref) <= TOL
        layer.close()


@pytest.mark.parametrize("M", [2048, 2051])
@pytest.mark.parametrize("fmt", ["w4g32", "w4c"])
def test_fp16_prefill_whole_output_two_kernels_agree(fmt, M):
    """Gemma2-2B gate+up shape at M = 2048 and at a ragged M whose last token tile is almost all
    padding (several rounds of workgroups per compute unit): the
    whole output of the kernel that converts weights in registers against the whole output of the
    kernel that writes dequantized weights to LDS (different pipelines, different summation
    orders: each is within the tolerance of the exact result, so they agree within twice that),
    and a sample of it against the oracle."""
    print(f"fp16 prefill whole output {fmt} M={M}", flush=True)
    rng = np.random.default_rng(77)
    fc = synth.FC("t", 2304, 18432, fmt)
    wq, s = synth.weights(4300, M, 0, fc)
    x = synth.activations(4300, M, 0, M, fc.K)
    layer = _layer(wq, s, fmt, max_m=M)
    xd = torch.from_numpy(x).to(DEV)
    for rep in range(3):
        y = layer.forward(xd)
        binding.qfc_tune(2, 9)
        try:
            y_other = layer.forward(xd)
        finally:
            binding.qfc_tune(2, 0)
        torch.cuda.synchronize()
        a, b = y.float(), y_other.float()
        rho = b.pow(2).mean(dim=1, keepdim=True).sqrt()
        err = ((a - b).abs() / torch.maximum(b.abs(), rho)).max().item()
        assert err <= 2 * TOL, err
    rows = np.sort(rng.choice(M, size=16, replace=False))
    cols = np.sort(rng.choice(fc.N, size=512, replace=False))
    ref = oracle.fc_weight_only(x[rows], wq[cols], s[cols], _group(fmt))
    assert _E(y.cpu().numpy()[np.ix_(rows, cols)], ref) <= TOL
    layer.close()


@pytest.mark.parametrize("form", [31, 32, 33, 34, 35, 36, 37])
@pytest.mark.parametrize("fmt", ["w4g32", "w4c", "w8c"])
def test_fp16_tiles_of_every_form(form, fmt):
    """The main kernel with binary16 activations in each of its forms (32 to 128 token rows per workgroup, K in one piece or two): one
    step of K, an odd number of steps (uneven halves), more than eight (a second unit of group scales); token rows one past a tile and
    one short of it; channels whose rows are aligned to 16, 8, 4 and 2 bytes; residual; gated output over whole and ragged channel tiles, even and
    uneven halves of K."""
    step = 64 if fmt == "w8c" else 128
    for M, N, steps in ((9, 70, 1), (33, 264, 2), (95, 300, 3), (129, 517, 5), (127, 90, 9), (161, 256, 10), (255, 1, 4), (97, 288, 5), (40, 96, 3), (130, 544, 9)):
        K = step * steps
        if form >= 35 and K < 256:
            continue  # (K in two halves is built for 256 and more; the number would leave the choice to the dispatch)
        print(f"fp16 tiles form={form} {fmt} M={M} N={N} K={K}", flush=True)
        wq, s = synth.weights(4500, M, N, synth.FC("t", K, N, fmt))
        x = synth.activations(4500, M, N, M, K)
        res = synth.activations(4500, M, N + 1, M, N)
        layer = _layer(wq, s, fmt, max_m=M, mode=binding.QFC_COMPUTE_FP16_DEQUANT)
        ref = oracle.fc_weight_only(x, wq, s, _group(fmt))
        xd, rd = torch.from_numpy(x).to(DEV), torch.from_numpy(res).to(DEV)
        guard = torch.full((M + 1, N), 77.0, dtype=torch.float16, device=DEV)
        binding.qfc_tune(2, form)
        try:
            binding.qfc_forward(layer.handle, xd, guard[:M])
            plain = guard[:M].cpu().numpy()
            binding.qfc_forward_fused(layer.handle, xd, guard[:M], residual=rd)
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(2, 0)
        assert _E(plain, ref) <= TOL, (M, N, K)
        assert _E(guard[:M].cpu().numpy(), ref + res.astype(np.float64)) <= TOL, (M, N, K)
        assert bool((guard[M] == 77.0).all())
        layer.close()
        if fmt == "w8c" or N % 32 != 0:
            continue
        x = (x * np.float16(0.25)).astype(np.float16)
        gated = binding.QuantLinear(wq, s, fmt, compute_mode=binding.QFC_COMPUTE_FP16_DEQUANT, max_m=M, gated_pairs=True)
        guard = torch.full((M + 1, N // 2), 77.0, dtype=torch.float16, device=DEV)
        binding.qfc_tune(2, form)
        try:
            binding.qfc_forward_fused(gated.handle, torch.from_numpy(x).to(DEV), guard[:M], activation=binding.QFC_ACT_SILU, gated_output=True)
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(2, 0)
        # (group scales: the product of two outputs that each carry the rounding of scaled weights, twice the tolerance)
        assert _E(guard[:M].cpu().numpy(), oracle.gated_output(oracle.fc_weight_only(x, wq, s, _group(fmt)), oracle.SILU)) <= (2 if fmt == "w4g32" else 1) * TOL
        assert bool((guard[M] == 77.0).all())
        gated.close()


# ------------------------------------------------------------------ decode with 8-bit activations (the paper's decode design)
@pytest.mark.parametrize("fmt", ["w8c", "w4c"])
@pytest.mark.parametrize("N,K", DECODE_SHAPES)
def test_decode_int8_activations(fmt, N, K):
    """Activations quantized inside the decode kernel: integer sums bit for bit (through the
    entry points that take quantized activations), y within tolerance of the step-by-step
    oracle, and the fused kernel equal to the pre-quantized one bit for bit."""
    fc = synth.FC("t", K, N, fmt)
    wq, sw = synth.weights(2100, N, K, fc)
    wq.flat[0] = -128 if fmt == "w8c" else -8
    layer = _layer(wq, sw, fmt, mode=binding.QFC_COMPUTE_INT8_ACT_DECODE)
    for M in range(1, 9):
        print(f"decode int8 activations {fmt} N={N} K={K} M={M}", flush=True)
        x = synth.activations(2100, N, K + M, M, K)
        if M == 3:
            x[1] = 0  # an all-zero token row: scale 0, codes 0, output 0
        xq_ref, sx_ref, acc_ref, y_ref = oracle.fc_int8_act(x, wq, sw)
        xq_d = torch.from_numpy(xq_ref).to(DEV)
        acc = torch.empty((M, N), dtype=torch.int32, device=DEV)
        binding.qfc_forward_acc_i32(layer.handle, xq_d, acc)
        y_q8 = torch.empty((M, N), dtype=torch.float16, device=DEV)
        binding.qfc_forward_q8(layer.handle, xq_d, torch.from_numpy(sx_ref).to(DEV), y_q8)
        y = _forward(layer, x)
        assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), M
        assert _E(y, y_ref) <= TOL, M
        assert np.array_equal(y.view(np.uint16), y_q8.cpu().numpy().view(np.uint16)), M
    layer.close()


def test_decode_int8_activations_llama_shapes_sampled():
    rng = np.random.default_rng(31)
    for i, fc in enumerate(synth.LLAMA_FCS_W4C):
        print(f"int8-activation decode {fc.name} {fc.K}->{fc.N}", flush=True)
        wq, sw = synth.weights(1103, 0, i, fc)
        x = synth.activations(1103, 0, i, 4, fc.K)
        layer = _layer(wq, sw, fc.fmt, mode=binding.QFC_COMPUTE_INT8_ACT_DECODE)
        y = _forward(layer, x)
        cols = np.sort(rng.choice(fc.N, size=512, replace=False))
        cols[0], cols[-1] = 0, fc.N - 1
        _, _, _, y_ref = oracle.fc_int8_act(x, wq[cols], sw[cols])
        assert _E(y[:, cols], y_ref) <= TOL
        layer.close()


# ------------------------------------------------------------------ A7 dispatch, batches, streams
@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
def test_dispatch_boundary_m8_m9(fmt):
    """M = 8 takes the decode kernel, M = 9 the prefill path: both within tolerance of the
    oracle, and the first eight rows of the M = 9 result agree with the M = 8 result to
    within twice the tolerance (different kernels, same definition)."""
    print(f"dispatch boundary {fmt}", flush=True)
    fc = synth.FC("t", 1024, 520, fmt)
    wq, s = synth.weights(7000, 0, 0, fc)
    x = synth.activations(7000, 0, 0, 9, fc.K)
    layer = _layer(wq, s, fmt, max_m=9)
    y8 = _forward(layer, x[:8])
    y9 = _forward(layer, x)
    if fmt == "w8c":
        _, _, _, ref9 = oracle.fc_int8_act(x, wq, s)
    else:
        ref9 = oracle.fc_weight_only(x, wq, s, _group(fmt))
    ref8 = oracle.fc_weight_only(x[:8], wq, s, _group(fmt))
    assert _E(y8, ref8) <= TOL
    assert _E(y9, ref9) <= TOL
    if fmt != "w8c":
        assert _E(y9[:8], ref8) <= TOL
    layer.close()


def test_forward_batch_equals_single_calls_on_a_side_stream():
    print("forward batch", flush=True)
    fcs = [synth.FC("a", 512, 300, "w4g32"), synth.FC("b", 2304, 264, "w4g32"), synth.FC("c", 256, 1000, "w8c")]
    layers, xs, singles = [], [], []
    for i, fc in enumerate(fcs):
        wq, s = synth.weights(7001, 0, i, fc)
        layers.append(_layer(wq, s, fc.fmt))
        xs.append(torch.from_numpy(synth.activations(7001, 0, i, 3, fc.K)).to(DEV))
        singles.append(layers[-1].forward(xs[-1]))
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    ys = [torch.full((3, l.N), 7.0, dtype=torch.float16, device=DEV) for l in layers]
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        fb = binding.ForwardBatch([l.handle for l in layers], xs, ys, 3)
        fb.run()
    side.synchronize()
    for y, y1 in zip(ys, singles):
        assert torch.equal(y.view(torch.int16), y1.view(torch.int16))
    for l in layers:
        l.close()


@pytest.mark.parametrize("fmt,M", [("w8c", 200), ("w4g32", 300), ("w4c", 300)])
def test_prefill_is_deterministic(fmt, M):
    print(f"prefill determinism {fmt}", flush=True)
    fc = synth.FC("t", 1152, 520, fmt)
    wq, s = synth.weights(7002, 0, 0, fc)
    x = synth.activations(7002, 0, 0, M, fc.K)
    layer = _layer(wq, s, fmt, max_m=M)
    y1 = _forward(layer, x)
    y2 = _forward(layer, x)
    assert np.array_equal(y1.view(np.uint16), y2.view(np.uint16))
    layer.close()


def test_error_paths_on_device():
    print("error paths", flush=True)
    fc = synth.FC("t", 64, 64, "w4g32")
    wq, s = synth.weights(6000, 0, 0, fc)
    layer = _layer(wq, s, "w4g32")
    x = torch.zeros((2, 64), dtype=torch.float16, device=DEV)
    xq = torch.zeros((2, 64), dtype=torch.int8, device=DEV)
    acc = torch.zeros((2, 64), dtype=torch.int32, device=DEV)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_forward_acc_i32(layer.handle, xq, acc)  # int8 product needs int8 per-channel weights
    assert e.value.code == 2
    small = torch.zeros(256, dtype=torch.uint8, device=DEV)
    big = synth.FC("t", 512, 64, "w8c")
    wq2, s2 = synth.weights(6001, 0, 0, big)
    layer2 = _layer(wq2, s2, "w8c")
    binding.qfc_bind_workspace(layer2.handle, small)
    with pytest.raises(binding.QfcError) as e:  # int8 prefill needs room for the quantized activations
        binding.qfc_forward(layer2.handle, torch.zeros((16, 512), dtype=torch.float16, device=DEV),
                            torch.zeros((16, 64), dtype=torch.float16, device=DEV))
    assert e.value.code == 3
    layer.close()
    layer2.close()
    del x


def test_binding_rejects_tensors_the_abi_cannot_check():
    """The C ABI takes pointers and row counts; the binding refuses tensors whose dtype, strides or
    dimensions do not match the handle before anything is launched."""
    fc = synth.FC("t", 128, 64, "w4g32")
    wq, s = synth.weights(6100, 0, 0, fc)
    layer = _layer(wq, s, "w4g32")
    x = torch.zeros((2, 128), dtype=torch.float16, device=DEV)
    y = torch.zeros((2, 64), dtype=torch.float16, device=DEV)
    binding.qfc_forward(layer.handle, x, y)
    bad = [(torch.zeros((2, 96), dtype=torch.float16, device=DEV), y),       # K of x
           (x, torch.zeros((2, 32), dtype=torch.float16, device=DEV)),       # N of y
           (x, torch.zeros((3, 64), dtype=torch.float16, device=DEV)),       # M of y
           (x.float(), y), (x, y.float()),                                   # dtypes
           (torch.zeros((2, 256), dtype=torch.float16, device=DEV)[:, ::2], y),  # strided view
           (x.cpu(), y)]
    for xb, yb in bad:
        with pytest.raises(ValueError):
            binding.qfc_forward(layer.handle, xb, yb)
        with pytest.raises(ValueError):
            binding.qfc_forward_fused(layer.handle, xb, yb)
    with pytest.raises(ValueError):
        binding.ForwardBatch([layer.handle], [x], [torch.zeros((2, 32), dtype=torch.float16, device=DEV)], 2)
    with pytest.raises(ValueError):
        binding.qfc_quantize_activations(x, torch.zeros((2, 64), dtype=torch.int8, device=DEV),
                                         torch.zeros((2,), dtype=torch.float32, device=DEV))
    layer.close()
    with pytest.raises(ValueError):
        binding.qfc_forward(ctypes.c_void_p(12345), x, y)  # not a live handle of this binding
    torch.cuda.synchronize()


# ------------------------------------------------------------------ element-wise operators fused with the layer
def _fused(layer, x, gate=None, act=binding.QFC_ACT_SILU, residual=None, alias=False):
    xd = torch.from_numpy(x).to(DEV)
    gd = torch.from_numpy(gate).to(DEV) if gate is not None else None
    rd = torch.from_numpy(residual).to(DEV) if residual is not None else None
    y = rd if alias else torch.empty((x.shape[0], layer.N), dtype=torch.float16, device=DEV)
    binding.qfc_forward_fused(layer.handle, xd, y, gate=gd, activation=act, residual=rd)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def _fused_ref(x, wq, s, fmt, gate, act, residual, int8_act=False):
    # (int8 activations: the gated input goes on to decide the row maximum and every 8-bit code, so
    # the reference takes it in binary32 like the quantizer; otherwise in fp64)
    gated = oracle.gated_input_f32 if int8_act else oracle.gated_input
    x_in = gated(gate, x, act) if gate is not None else x
    ref = oracle.fc_int8_act(x_in, wq, s)[3] if int8_act else oracle.fc_weight_only(x_in, wq, s, _group(fmt))
    return oracle.add_residual(ref, residual) if residual is not None else ref


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(17, 96), (130, 256), (1000, 2304), (96, 14336)])
def test_decode_fused_gate_and_residual(fmt, N, K):
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3100, N, K, fc)
    layer = _layer(wq, s, fmt)
    for M in (1, 2, 3, 5, 8):
        print(f"decode fused {fmt} N={N} K={K} M={M}", flush=True)
        up = synth.activations(3100, N, K + M, M, K)
        gate = synth.activations(3101, N, K + M, M, K)
        res = synth.activations(3102, N, K + M, M, N)
        if M == 3:
            gate[1] = 0  # act(0) = 0: the row's input is zero, the output is the residual
        act = binding.QFC_ACT_SILU if M % 2 else binding.QFC_ACT_GELU_TANH
        oact = oracle.SILU if M % 2 else oracle.GELU_TANH
        y = _fused(layer, up, gate, act, res)
        assert _E(y, _fused_ref(up, wq, s, fmt, gate, oact, res)) <= TOL, M
        if M == 3:
            assert np.array_equal(y[1], res[1])
        # each part alone, and the output written over the residual
        y = _fused(layer, up, gate, act, None)
        assert _E(y, _fused_ref(up, wq, s, fmt, gate, oact, None)) <= TOL, M
        y = _fused(layer, up, None, act, res, alias=True)
        assert _E(y, _fused_ref(up, wq, s, fmt, None, oact, res)) <= TOL, M
        # no parts: the plain call, bit for bit
        assert np.array_equal(_fused(layer, up), _forward(layer, up))
    layer.close()


def test_decode_fused_gate_matches_the_unfused_pipeline():
    """fp16(act(gate) * up) computed on the host in fp32 and fed to the plain call gives the same
    bits as the fused call whenever the two fp32 evaluations round to the same binary16 value;
    with the oracle's binary16 input instead, the outputs agree within the tolerance."""
    fc = synth.FC("t", 2048, 512, "w4g32")
    wq, s = synth.weights(3200, 0, 0, fc)
    layer = _layer(wq, s, "w4g32")
    up = synth.activations(3200, 0, 1, 4, fc.K)
    gate = synth.activations(3200, 0, 2, 4, fc.K)
    x_in = oracle.gated_input(gate, up, oracle.SILU)
    y_fused = _fused(layer, up, gate, binding.QFC_ACT_SILU)
    y_plain = _forward(layer, x_in)
    assert _E(y_fused, y_plain.astype(np.float64)) <= 1e-3
    layer.close()


@pytest.mark.parametrize("M,N,K", [(9, 1, 32), (100, 130, 96), (200, 300, 512), (300, 1000, 2304)])
def test_int8_prefill_fused_gate_and_residual(M, N, K):
    print(f"int8 prefill fused M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, "w8c")
    wq, sw = synth.weights(3300, M, N, fc)
    up = synth.activations(3300, M, N, M, K)
    gate = synth.activations(3301, M, N, M, K)
    res = synth.activations(3302, M, N, M, N)
    gate[M // 2] = 0
    layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    for act, oact in ((binding.QFC_ACT_SILU, oracle.SILU), (binding.QFC_ACT_GELU_TANH, oracle.GELU_TANH)):
        y = _fused(layer, up, gate, act, res)
        ref = _fused_ref(up, wq, sw, "w8c", gate, oact, res, int8_act=True)
        # the quantizer evaluates the gate activation with the library exponential and an IEEE
        # division (fp32 within a few units in the last place of the real value), so the binary16
        # input and the 8-bit codes are the definition's
        e = _E(y, ref)
        print(f"  act {act}: E = {e:.3e}", flush=True)
        assert e <= TOL
        assert np.array_equal(y[M // 2], res[M // 2])
    y = _fused(layer, up, None, 0, res)
    assert _E(y, _fused_ref(up, wq, sw, "w8c", None, 0, res, int8_act=True)) <= TOL
    assert np.array_equal(_fused(layer, up), _forward(layer, up))
    layer.close()


@pytest.mark.parametrize("fmt", ["w4g32", "w4c"])
@pytest.mark.parametrize("M,N,K", [(9, 1, 32), (100, 130, 96), (130, 1000, 2304), (300, 264, 128), (129, 520, 1152)])
def test_fp16_prefill_fused_residual(fmt, M, N, K):
    print(f"fp16 prefill residual {fmt} M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3400, M, N, fc)
    x = synth.activations(3400, M, N, M, K)
    res = synth.activations(3401, M, N, M, N)
    layer = _layer(wq, s, fmt, max_m=M)
    y = _fused(layer, x, None, 0, res)
    assert _E(y, _fused_ref(x, wq, s, fmt, None, 0, res)) <= TOL
    assert np.array_equal(_fused(layer, x), _forward(layer, x))
    with pytest.raises(binding.QfcError) as e:  # no place for the gate on this path
        _fused(layer, x, x, binding.QFC_ACT_SILU, None)
    assert e.value.code == binding.QFC_ERR_UNSUPPORTED
    layer.close()


def test_fused_mlp_llama_shapes_sampled():
    """down(silu(gate) * up) + residual at the full Llama-3.1-8B shape (K = 14336 -> N = 4096)."""
    fc = synth.LLAMA_FCS_W4[3]
    wq, s = synth.weights(1003, 0, 3, fc)
    layer = _layer(wq, s, fc.fmt)
    rng = np.random.default_rng(31)
    for M in (1, 4):
        up = synth.activations(1003, 0, 30, M, fc.K)
        gate = synth.activations(1003, 0, 31, M, fc.K)
        res = synth.activations(1003, 0, 32, M, fc.N)
        y = _fused(layer, up, gate, binding.QFC_ACT_SILU, res)
        cols = np.sort(rng.choice(fc.N, size=256, replace=False))
        cols[0], cols[-1] = 0, fc.N - 1
        ref = _fused_ref(up, wq[cols], s[cols], fc.fmt, gate, oracle.SILU, res[:, cols])
        assert _E(y[:, cols], ref) <= TOL
    layer.close()


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(32, 96), (160, 256), (2048, 2304), (64, 14336)])
def test_decode_gated_output(fmt, N, K):
    """The layer produces [gate; other]; y [M, N/2] = fp16(act(gate) * other) from the unrounded sums."""
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3500, N, K, fc)
    layer = _layer(wq, s, fmt)
    for M in (1, 2, 3, 4, 7, 8):
        print(f"decode gated output {fmt} N={N} K={K} M={M}", flush=True)
        # small activations: the product of two outputs must stay inside the binary16 range
        x = (synth.activations(3500, N, K + M, M, K) * np.float16(0.0625)).astype(np.float16)
        act, oact = (binding.QFC_ACT_SILU, oracle.SILU) if M % 2 else (binding.QFC_ACT_GELU_TANH, oracle.GELU_TANH)
        xd = torch.from_numpy(x).to(DEV)
        y = torch.full((M, N // 2), 77.0, dtype=torch.float16, device=DEV)
        binding.qfc_forward_fused(layer.handle, xd, y, activation=act, gated_output=True)
        torch.cuda.synchronize()
        ref = oracle.gated_output(oracle.fc_weight_only(x, wq, s, _group(fmt)), oact)
        assert _E(y.cpu().numpy(), ref) <= TOL, M
    # combinations the interface excludes
    xd = torch.from_numpy(synth.activations(3500, N, K, 1, K)).to(DEV)
    y = torch.empty((1, N // 2), dtype=torch.float16, device=DEV)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_forward_fused(layer.handle, xd, y, residual=y, gated_output=True)
    assert e.value.code == binding.QFC_ERR_INVALID_ARG
    layer.close()


# Layers packed in pairs (the row tiles of the two branches interleaved): the merged gating in every kernel
@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(32, 32), (160, 96), (1024, 256), (2080, 1152)])
def test_paired_packing_round_trip_and_decode(fmt, N, K):
    print(f"paired packing {fmt} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3600, N, K, fc)
    layer = binding.QuantLinear(wq, s, fmt, gated_pairs=True)
    plain = binding.QuantLinear(wq, s, fmt)
    # the logical interface does not change: unpack returns what pack was given
    wq_back = torch.empty((N, K), dtype=torch.int8, device=DEV)
    s_back = torch.empty_like(torch.as_tensor(s)).to(DEV)
    binding.qfc_unpack_weights(layer.handle, wq_back, s_back)
    torch.cuda.synchronize()
    assert np.array_equal(wq_back.cpu().numpy(), wq)
    assert np.array_equal(s_back.cpu().numpy().view(np.uint8), np.ascontiguousarray(s).view(np.uint8))
    # and the packed bytes are a permutation of the plain packing's row tiles
    a, b = layer.packed.cpu().numpy(), plain.packed.cpu().numpy()
    assert a.shape == b.shape and (N == 32 or not np.array_equal(a, b))  # (two row tiles: nothing to interleave)
    for M in (1, 3, 8):
        x = (synth.activations(3600, N, K + M, M, K) * np.float16(0.0625)).astype(np.float16)
        xd = torch.from_numpy(x).to(DEV)
        act, oact = (binding.QFC_ACT_SILU, oracle.SILU) if M % 2 else (binding.QFC_ACT_GELU_TANH, oracle.GELU_TANH)
        y = torch.full((M, N // 2), 77.0, dtype=torch.float16, device=DEV)
        y_plain = torch.empty_like(y)
        binding.qfc_forward_fused(layer.handle, xd, y, activation=act, gated_output=True)
        binding.qfc_forward_fused(plain.handle, xd, y_plain, activation=act, gated_output=True)
        torch.cuda.synchronize()
        ref = oracle.gated_output(oracle.fc_weight_only(x, wq, s, _group(fmt)), oact)
        assert _E(y.cpu().numpy(), ref) <= TOL, M
        # same row tiles in the same order, wherever they sit in memory: the same bits
        assert np.array_equal(y.cpu().numpy().view(np.uint16), y_plain.cpu().numpy().view(np.uint16)), M
    # a layer packed in pairs only computes the gated output
    xd = torch.from_numpy(synth.activations(3600, N, K, 2, K)).to(DEV)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_forward(layer.handle, xd, torch.empty((2, N), dtype=torch.float16, device=DEV))
    assert e.value.code == binding.QFC_ERR_UNSUPPORTED
    layer.close()
    plain.close()


@pytest.mark.parametrize("fmt,mode", [("w8c", None), ("w4c", binding.QFC_COMPUTE_INT8_ACT), ("w4g32", None), ("w4c", None)])
@pytest.mark.parametrize("M,N,K", [(9, 32, 128), (100, 160, 384), (130, 1024, 256), (300, 2080, 1152), (513, 544, 2304)])
def test_prefill_gated_output(fmt, mode, M, N, K):
    """act(gate) * up in the store phase of the kernels that the sizes lead to (layer packed in pairs; with int8 activations those for few
    token rows) against the oracle: the element-wise product of the two halves of the unrounded outputs."""
    print(f"prefill gated output {fmt} mode={mode} M={M} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3700, M, N, fc)
    x = (synth.activations(3700, M, N, M, K) * np.float16(0.125)).astype(np.float16)
    layer = binding.QuantLinear(wq, s, fmt, compute_mode=mode, max_m=M, gated_pairs=True)
    int8 = fmt == "w8c" or mode == binding.QFC_COMPUTE_INT8_ACT
    full = oracle.fc_int8_act(x, wq, s)[3] if int8 else oracle.fc_weight_only(x, wq, s, _group(fmt))
    xd = torch.from_numpy(x).to(DEV)
    for act, oact in ((binding.QFC_ACT_SILU, oracle.SILU), (binding.QFC_ACT_GELU_TANH, oracle.GELU_TANH)):
        y = torch.full((M, N // 2), 77.0, dtype=torch.float16, device=DEV)
        binding.qfc_forward_fused(layer.handle, xd, y, activation=act, gated_output=True)
        torch.cuda.synchronize()
        e = _E(y.cpu().numpy(), oracle.gated_output(full, oact))
        print(f"  act {act}: E = {e:.3e}", flush=True)
        # the product of two outputs, each within the bound of its own path (the fp16 path with group
        # scales folded into the weights carries ~1e-3 per factor)
        assert e <= (2 * TOL if fmt == "w4g32" else TOL)
    layer.close()


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(32, 96), (160, 1152), (224, 2304)])
def test_decode_gated_output_two_pairs_per_workgroup(fmt, N, K):
    """Decode workgroups that take two pairs of row tiles (the last one may own one): the same bits as with one
    pair, both packings, with and without the merged normalization, whole and half units; and the oracle."""
    print(f"two pairs {fmt} N={N} K={K}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3650, N, K, fc)
    gamma = (synth.activations(3651, N, K, 1, K)[0] * np.float16(0.25)).astype(np.float16)
    gd = torch.from_numpy(gamma).to(DEV)
    for paired in (False, True):
        layer = binding.QuantLinear(wq, s, fmt, gated_pairs=paired)
        for M in (1, 2, 3, 4, 5, 7, 8):
            x = (synth.activations(3650, N, K + M, M, K) * np.float16(0.0625)).astype(np.float16)
            xd = torch.from_numpy(x).to(DEV)
            for norm in (False, True):
                kw = dict(norm_gamma=gd, norm_eps=1e-5) if norm else {}
                for half in (0, 1):
                    ys = []
                    for pairs in (1, 2):
                        binding.qfc_tune(4, half)
                        binding.qfc_tune(10, pairs)
                        try:
                            y = torch.full((M, N // 2), 77.0, dtype=torch.float16, device=DEV)
                            binding.qfc_forward_fused(layer.handle, xd, y, activation=binding.QFC_ACT_SILU, gated_output=True, **kw)
                            torch.cuda.synchronize()
                        finally:
                            binding.qfc_tune(4, -1)
                            binding.qfc_tune(10, 0)
                        ys.append(y.cpu().numpy())
                    assert np.array_equal(ys[0].view(np.uint16), ys[1].view(np.uint16)), (paired, M, norm, half)
                if norm:
                    full = oracle.rms_scale(x, 1e-5)[:, None] * oracle.fc_weight_only(oracle.norm_weighted_input(x, gamma, 0.0), wq, s, _group(fmt))
                else:
                    full = oracle.fc_weight_only(x, wq, s, _group(fmt))
                assert _E(ys[1], oracle.gated_output(full, oracle.SILU)) <= TOL, (paired, M, norm)
        layer.close()


def test_prefill_gated_output_llama_gate_up_sampled():
    """The gate+up layer of Llama-3.1-8B at M = 1024 (int8 activations, 8-bit and 4-bit per-channel weights)
    and of Gemma2-2B at M = 2048 (fp16, int4 group-32), packed in pairs: sampled rows and channels
    against the oracle."""
    rng = np.random.default_rng(46)
    for fc, M, seed, mode in ((synth.LLAMA_FCS_W8[2], 1024, 1004, None), (synth.GEMMA_FCS_W4[2], 2048, 1005, None),
                              (synth.LLAMA_FCS_W4C[2], 1024, 1104, binding.QFC_COMPUTE_INT8_ACT)):
        print(f"prefill gated output {fc.name} {fc.fmt} {fc.K}->{fc.N} M={M}", flush=True)
        wq, s = synth.weights(seed, 0, 2, fc)
        x = (synth.activations(seed, 0, 2, M, fc.K) * np.float16(0.125)).astype(np.float16)
        layer = binding.QuantLinear(wq, s, fc.fmt, compute_mode=mode, max_m=M, gated_pairs=True)
        y = torch.empty((M, fc.N // 2), dtype=torch.float16, device=DEV)
        binding.qfc_forward_fused(layer.handle, torch.from_numpy(x).to(DEV), y, activation=binding.QFC_ACT_SILU,
                                  gated_output=True)
        torch.cuda.synchronize()
        half = fc.N // 2
        rows = np.sort(rng.choice(M, size=32, replace=False))
        cols = np.sort(rng.choice(half, size=256, replace=False))
        rows[0], rows[-1], cols[0], cols[-1] = 0, M - 1, 0, half - 1
        both = np.concatenate([cols, cols + half])
        if fc.fmt == "w8c" or mode == binding.QFC_COMPUTE_INT8_ACT:
            full = oracle.fc_int8_act(x[rows], wq[both], s[both])[3]
        else:
            full = oracle.fc_weight_only(x[rows], wq[both], s[both], 32)
        ref = oracle.gated_output(full, oracle.SILU)
        assert _E(y.cpu().numpy()[np.ix_(rows, cols)], ref) <= (2 * TOL if fc.fmt == "w4g32" else TOL)
        layer.close()


def test_paired_packing_restrictions():
    fc = synth.FC("t", 96, 64, "w8c")
    wq, s = synth.weights(3800, 0, 0, fc)
    with pytest.raises(binding.QfcError) as e:  # the halves must be whole row tiles
        binding.QuantLinear(wq[:48], s[:48], "w8c", gated_pairs=True)
    assert e.value.code == binding.QFC_ERR_INVALID_ARG
    layer = binding.QuantLinear(wq, s, "w8c", max_m=16, gated_pairs=True)
    plain = binding.QuantLinear(wq, s, "w8c", max_m=16)
    x = torch.zeros((16, 96), dtype=torch.float16, device=DEV)
    xq = torch.zeros((16, 96), dtype=torch.int8, device=DEV)
    sx = torch.zeros((16,), dtype=torch.float32, device=DEV)
    y = torch.zeros((16, 64), dtype=torch.float16, device=DEV)
    yh = torch.zeros((16, 32), dtype=torch.float16, device=DEV)
    for call in (lambda: binding.qfc_forward(layer.handle, x, y),
                 lambda: binding.qfc_forward_q8(layer.handle, xq, sx, y),
                 lambda: binding.qfc_forward_acc_i32(layer.handle, xq, torch.zeros((16, 64), dtype=torch.int32, device=DEV)),
                 lambda: binding.qfc_embedding(layer.handle, torch.zeros(2, dtype=torch.int32, device=DEV),
                                               torch.zeros((2, 96), dtype=torch.float16, device=DEV)),
                 # gated output at M > 8 needs the paired packing
                 lambda: binding.qfc_forward_fused(plain.handle, x, yh, gated_output=True)):
        with pytest.raises(binding.QfcError) as e:
            call()
        assert e.value.code == binding.QFC_ERR_UNSUPPORTED
    binding.qfc_forward_fused(layer.handle, x, yh, gated_output=True)  # (and works with it)
    # the fp16 path's merged gating needs K to be a multiple of 128
    fc4 = synth.FC("t", 96, 64, "w4g32")
    wq4, s4 = synth.weights(3801, 0, 0, fc4)
    l4 = binding.QuantLinear(wq4, s4, "w4g32", max_m=16, gated_pairs=True)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_forward_fused(l4.handle, x, yh, gated_output=True)
    assert e.value.code == binding.QFC_ERR_UNSUPPORTED
    torch.cuda.synchronize()
    for l in (layer, plain, l4):
        l.close()


def test_gated_output_needs_even_halves_of_whole_tiles():
    fc = synth.FC("t", 64, 48, "w8c")  # N / 2 = 24 is not a whole number of 16-row tiles
    wq, s = synth.weights(3501, 0, 0, fc)
    layer = _layer(wq, s, "w8c")
    xd = torch.from_numpy(synth.activations(3501, 0, 0, 1, 64)).to(DEV)
    y = torch.empty((1, 24), dtype=torch.float16, device=DEV)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_forward_fused(layer.handle, xd, y, gated_output=True)
    assert e.value.code == binding.QFC_ERR_INVALID_ARG
    layer.close()


# ------------------------------------------------------------------ RMS normalization with merged residual and quantization
@pytest.mark.parametrize("M,K", [(1, 32), (3, 96), (5, 2304), (8, 4096), (70, 4096), (33, 14336), (600, 256)])
def test_rmsnorm_residual_quantize(M, K):
    print(f"rmsnorm M={M} K={K}", flush=True)
    x = synth.activations(3600, M, K, M, K)
    r = synth.activations(3601, M, K, M, K)
    gamma = (synth.activations(3602, M, K, 1, K)[0] * np.float16(0.25)).astype(np.float16)
    if M > 2:
        x[1] = 0
        r[1] = 0  # an all-zero row: h = 0, y = 0 (eps > 0), codes 0, scale 0
    xd, rd, gd = (torch.from_numpy(t).to(DEV) for t in (x, r, gamma))
    for goff, eps in ((0.0, 1e-5), (1.0, 1e-6)):
        h_out = torch.empty((M, K), dtype=torch.float16, device=DEV)
        y = torch.empty((M, K), dtype=torch.float16, device=DEV)
        xq = torch.empty((M, K), dtype=torch.int8, device=DEV)
        sx = torch.empty((M,), dtype=torch.float32, device=DEV)
        binding.qfc_rmsnorm(xd, gd, eps, goff, residual=rd, h_out=h_out, y=y, xq=xq, sx=sx)
        torch.cuda.synchronize()
        h_ref, y_ref = oracle.rmsnorm(x, gamma, eps, goff, residual_f16=r)
        # the residual stream: one correctly rounded binary16 addition, bit for bit
        assert np.array_equal(h_out.cpu().numpy().view(np.uint16), h_ref.view(np.uint16))
        y_gpu = y.cpu().numpy()
        assert _E(y_gpu, y_ref) <= TOL
        # the quantization is the activation quantization of the stored y, bit for bit
        xq_ref, sx_ref = oracle.quantize_activations(y_gpu)
        assert np.array_equal(xq.cpu().numpy(), xq_ref)
        assert np.array_equal(sx.cpu().numpy().view(np.uint32), sx_ref.view(np.uint32))
        if M > 2:
            assert not y_gpu[1].any() and not xq_ref[1].any() and sx_ref[1] == 0
    # without a residual, and with only some outputs; in place on the residual stream
    y2 = torch.empty((M, K), dtype=torch.float16, device=DEV)
    binding.qfc_rmsnorm(xd, gd, 1e-5, 0.0, y=y2)
    torch.cuda.synchronize()
    h_ref, y_ref = oracle.rmsnorm(x, gamma, 1e-5, 0.0)
    assert _E(y2.cpu().numpy(), y_ref) <= TOL
    stream_buf = xd.clone()
    xq = torch.empty((M, K), dtype=torch.int8, device=DEV)
    sx = torch.empty((M,), dtype=torch.float32, device=DEV)
    binding.qfc_rmsnorm(stream_buf, gd, 1e-5, 0.0, residual=rd, h_out=stream_buf, xq=xq, sx=sx)
    torch.cuda.synchronize()
    h_ref, y_ref = oracle.rmsnorm(x, gamma, 1e-5, 0.0, residual_f16=r)
    assert np.array_equal(stream_buf.cpu().numpy().view(np.uint16), h_ref.view(np.uint16))
    # codes of the oracle's y agree except where the fp32 evaluation rounds y to the neighbouring binary16 value
    xq_o, sx_o = oracle.quantize_activations(y_ref.astype(np.float16))
    assert np.max(np.abs(xq.cpu().numpy().astype(np.int32) - xq_o.astype(np.int32))) <= 1
    assert np.allclose(sx.cpu().numpy(), sx_o, rtol=2e-3, atol=0)


def test_rmsnorm_feeds_the_int8_layer():
    """norm -> quantized activations -> qfc_forward_q8 equals norm -> y -> int8 prefill layer, bit for bit."""
    M, K, N = 40, 512, 300
    fc = synth.FC("t", K, N, "w8c")
    wq, sw = synth.weights(3700, M, N, fc)
    layer = _layer(wq, sw, "w8c", max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    x = torch.from_numpy(synth.activations(3700, M, N, M, K)).to(DEV)
    gamma = torch.from_numpy(synth.activations(3701, M, N, 1, K)[0]).to(DEV)
    y = torch.empty((M, K), dtype=torch.float16, device=DEV)
    xq = torch.empty((M, K), dtype=torch.int8, device=DEV)
    sx = torch.empty((M,), dtype=torch.float32, device=DEV)
    binding.qfc_rmsnorm(x, gamma, 1e-5, 0.0, y=y, xq=xq, sx=sx)
    out_a = torch.empty((M, N), dtype=torch.float16, device=DEV)
    out_b = torch.empty((M, N), dtype=torch.float16, device=DEV)
    binding.qfc_forward_q8(layer.handle, xq, sx, out_a)
    binding.qfc_forward(layer.handle, y, out_b)
    torch.cuda.synchronize()
    assert np.array_equal(out_a.cpu().numpy().view(np.uint16), out_b.cpu().numpy().view(np.uint16))
    layer.close()


@pytest.mark.parametrize("fmt", ["w8c", "w4c"])
@pytest.mark.parametrize("M,K,N", [(40, 512, 300), (300, 2304, 264), (1024, 4096, 512)])
def test_rmsnorm_writes_the_next_layers_tiled_activations(fmt, M, K, N):
    """The normalization as the producer of the int8 layer's input: qfc_rmsnorm(consumer = layer) leaves
    the codes in the layer's workspace in the order its product kernel reads, and qfc_forward_q8 on
    them (no pass over the activations in between) gives the bits of the two-step route, which in turn
    is within the tolerance of the oracle's norm -> quantize -> integer product -> rescale."""
    print(f"rmsnorm -> tiled activations {fmt} M={M} K={K} N={N}", flush=True)
    fc = synth.FC("t", K, N, fmt)
    wq, sw = synth.weights(3750, M, N, fc)
    layer = _layer(wq, sw, fmt, max_m=M, mode=binding.QFC_COMPUTE_INT8_ACT)
    xh = synth.activations(3750, M, N, M, K)
    rh = synth.activations(3751, M, N, M, K)
    gh = synth.activations(3752, M, N, 1, K)[0]
    x, r, gamma = (torch.from_numpy(t).to(DEV) for t in (xh, rh, gh))
    xq = torch.empty((M, K), dtype=torch.int8, device=DEV)
    sx = torch.empty((M,), dtype=torch.float32, device=DEV)
    h_a = torch.empty((M, K), dtype=torch.float16, device=DEV)
    h_b = torch.empty((M, K), dtype=torch.float16, device=DEV)
    out_a = torch.empty((M, N), dtype=torch.float16, device=DEV)
    out_b = torch.full((M, N), 9.0, dtype=torch.float16, device=DEV)
    binding.qfc_rmsnorm(x, gamma, 1e-5, 1.0, residual=r, h_out=h_a, xq=xq, sx=sx)
    binding.qfc_forward_q8(layer.handle, xq, sx, out_a)
    layer.workspace.fill_(0x55)  # whatever the first route left there
    binding.qfc_rmsnorm(x, gamma, 1e-5, 1.0, residual=r, h_out=h_b, consumer=layer.handle)
    binding.qfc_forward_q8(layer.handle, None, None, out_b)
    torch.cuda.synchronize()
    assert np.array_equal(h_a.cpu().numpy().view(np.uint16), h_b.cpu().numpy().view(np.uint16))
    assert np.array_equal(out_a.cpu().numpy().view(np.uint16), out_b.cpu().numpy().view(np.uint16))
    h_ref, y_ref = oracle.rmsnorm(xh, gh, 1e-5, 1.0, rh)
    assert np.array_equal(h_b.cpu().numpy().view(np.uint16), h_ref.view(np.uint16))
    # the layer's input is the stored (binary16) y; where the fp32 evaluation of y rounds to the other
    # neighbour the 8-bit code may move, so this last comparison is to the bound of the integer path
    ref = oracle.fc_int8_act(y_ref.astype(np.float16), wq, sw)[3]
    assert _E(out_b.cpu().numpy(), ref) <= 2 * TOL
    # both outputs at once (row-major codes and the tiled ones)
    xq2, sx2 = torch.empty_like(xq), torch.empty_like(sx)
    binding.qfc_rmsnorm(x, gamma, 1e-5, 1.0, residual=r, xq=xq2, sx=sx2, consumer=layer.handle)
    torch.cuda.synchronize()
    assert torch.equal(xq2, xq) and torch.equal(sx2, sx)
    # a decode-size M or a layer of another width is refused
    with pytest.raises(binding.QfcError):
        binding.qfc_rmsnorm(x[:4], gamma, 1e-5, 1.0, consumer=layer.handle)
    layer.close()


# ------------------------------------------------------------------ attention-side operators
def _attn_shape(B, h_q, h_kv, d, C):
    return binding.AttnShape(B, h_q, h_kv, d, C)


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,pos0", [(1, 1, 4, 2, 64, 64, 0), (2, 3, 8, 2, 128, 128, 17),
                                                   (1, 1, 32, 8, 128, 192, 131), (3, 2, 8, 4, 256, 64, 62),
                                                   (1, 1, 2, 1, 128, 131072, 131071)])
def test_rope_qkv_layout(B, S, h_q, h_kv, d, C, pos0):
    print(f"rope B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} C={C} pos0={pos0}", flush=True)
    base = 500000.0 if d == 128 else 10000.0
    W = (h_q + 2 * h_kv) * d
    qkv = synth.activations(3800, B, S, B * S, W).reshape(B, S, W)
    G, g = B * h_kv, h_q // h_kv
    shape = _attn_shape(B, h_q, h_kv, d, C)
    q_out = torch.zeros((G, S * g, d), dtype=torch.float16, device=DEV)
    # sentinels in the caches: nothing but the S new positions may change
    kc = torch.full((G, C, d), 3.0, dtype=torch.float16, device=DEV)
    vc = torch.full((G, C // 64, d, 64), 5.0, dtype=torch.float16, device=DEV)
    binding.qfc_rope_qkv(torch.from_numpy(qkv).to(DEV), pos0, shape, base, q_out, kc, vc)
    torch.cuda.synchronize()
    vc = binding.vcache_logical(vc)
    q_ref, k_ref, v_ref = oracle.rope_qkv_layout(qkv, pos0, h_q, h_kv, d, base)
    kc, vc = kc.cpu().numpy(), vc.cpu().numpy()

    def close(a, b):  # one binary16 unit in the last place of the larger magnitude, or of 2^-10
        a, b = a.astype(np.float64), b.astype(np.float64)
        return np.all(np.abs(a - b) <= 2.0 ** -10 * np.maximum(np.maximum(np.abs(a), np.abs(b)), 2.0 ** -10))

    assert close(q_out.cpu().numpy(), q_ref)
    assert close(kc[:, pos0:pos0 + S], k_ref)
    assert np.array_equal(vc[:, :, pos0:pos0 + S].view(np.uint16), v_ref.transpose(0, 2, 1).view(np.uint16))
    kc[:, pos0:pos0 + S] = 3.0
    vc[:, :, pos0:pos0 + S] = 5.0
    assert np.all(kc == 3.0) and np.all(vc == 5.0)


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,n_ctx", [(1, 1, 4, 4, 64, 64, 1), (1, 1, 4, 2, 64, 64, 33),
                                                    (2, 1, 32, 8, 128, 1024, 1000), (1, 1, 8, 4, 256, 4096, 4096),
                                                    (1, 4, 8, 2, 128, 512, 259), (3, 2, 16, 2, 128, 128, 65),
                                                    (1, 1, 16, 1, 64, 8192, 8191), (1, 1, 32, 8, 128, 16384, 12345)])
def test_attention_over_the_cache(B, S, h_q, h_kv, d, C, n_ctx):
    print(f"attention B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} C={C} n_ctx={n_ctx}", flush=True)
    G, g = B * h_kv, h_q // h_kv
    M = S * g
    rng = np.random.default_rng(n_ctx * 31 + d)
    q = rng.standard_normal((G, M, d)).astype(np.float16)
    K = rng.standard_normal((G, C, d)).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    # a few dominant keys, so that the softmax is not flat; and poison past the end of the context
    for gi in range(G):
        K[gi, rng.integers(0, n_ctx)] = (q[gi, 0].astype(np.float32) * 2).astype(np.float16)
    Kd, Vd = K.copy(), V.copy()
    Kd[:, n_ctx:] = np.float16(np.nan)
    Vd[:, :, n_ctx:] = np.float16(np.inf)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
    out = torch.full((G, M, d), 9.0, dtype=torch.float16, device=DEV)
    binding.qfc_attention(torch.from_numpy(q).to(DEV), torch.from_numpy(Kd).to(DEV), binding.vcache_physical(torch.from_numpy(Vd).to(DEV)), S,
                          n_ctx, shape, ws, out)
    torch.cuda.synchronize()
    ref = oracle.attention(q, K, V, n_ctx, S)
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got))
    assert _E(got.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL


# more KV heads than compute units: a last round of few workgroups (cut walks) and 13 steps, one fewer than that asks for
@pytest.mark.parametrize("B,d,n_ctx", [(65, 64, 897), (65, 64, 832), (86, 128, 900)])
def test_attention_many_heads_last_round_of_few(B, d, n_ctx):
    test_attention_over_the_cache(B, 1, 4, 4, d, 960, n_ctx)


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,n_ctx", [(1, 1, 4, 1, 64, 640, 577), (2, 1, 8, 2, 128, 704, 700), (1, 3, 4, 1, 256, 384, 321)])
def test_attention_any_number_of_workgroups_per_head(B, S, h_q, h_kv, d, C, n_ctx):
    """The combination of 1 to 64 partial results (whole and broken groups of eight), workgroups with one step for
    four wavefronts and with none; and the number the library picks."""
    print(f"attention splits B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} n_ctx={n_ctx}", flush=True)
    G, M = B * h_kv, S * (h_q // h_kv)
    rng = np.random.default_rng(n_ctx)
    q = rng.standard_normal((G, M, d)).astype(np.float16)
    K = rng.standard_normal((G, C, d)).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    K[:, 5] = (q[:, 0].astype(np.float32) * 2).astype(np.float16)
    ref = oracle.attention(q, K, V, n_ctx, S)
    K[:, n_ctx:] = np.float16(np.nan)
    V[:, :, n_ctx:] = np.float16(np.inf)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
    qd, kd, vd = torch.from_numpy(q).to(DEV), torch.from_numpy(K).to(DEV), binding.vcache_physical(torch.from_numpy(V).to(DEV))
    for splits in (0, 1, 2, 7, 8, 9, 11, 16, 17, 33, 63, 64):
        out = torch.full((G, M, d), 9.0, dtype=torch.float16, device=DEV)
        binding.qfc_tune(12, splits)
        try:
            binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, out)
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(12, 0)
        got = out.cpu().numpy()
        assert np.all(np.isfinite(got)), splits
        assert _E(got.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL, splits


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,n_ctx", [(1, 5, 8, 2, 64, 64, 5), (1, 40, 4, 4, 128, 128, 40),
                                                    (2, 33, 8, 2, 128, 192, 150), (1, 100, 8, 4, 256, 128, 100),
                                                    (1, 256, 32, 8, 128, 512, 300), (1, 64, 16, 1, 64, 1024, 1000),
                                                    (1, 1024, 32, 8, 128, 1024, 1024),
                                                    (1, 640, 8, 4, 256, 640, 640)])
def test_attention_many_query_rows(B, S, h_q, h_kv, d, C, n_ctx):
    """Prefill: more than 16 query rows per KV head, causal by token, ragged row and position counts."""
    print(f"prefill attention B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} C={C} n_ctx={n_ctx}", flush=True)
    G, g = B * h_kv, h_q // h_kv
    M = S * g
    assert M > 16
    rng = np.random.default_rng(n_ctx * 17 + S)
    q = rng.standard_normal((G, M, d)).astype(np.float16)
    K = rng.standard_normal((G, C, d)).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    Kd, Vd = K.copy(), V.copy()
    Kd[:, n_ctx:] = np.float16(np.nan)
    Vd[:, :, n_ctx:] = np.float16(np.inf)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
    out = torch.full((G, M, d), 9.0, dtype=torch.float16, device=DEV)
    qd, kd, vd = torch.from_numpy(q).to(DEV), torch.from_numpy(Kd).to(DEV), binding.vcache_physical(torch.from_numpy(Vd).to(DEV))
    binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, out)
    torch.cuda.synchronize()
    ref = oracle.attention(q, K, V, n_ctx, S)
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got))
    assert _E(got.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL
    # whole walks by one wavefront and by two, as launches of many blocks take them, and each of them twice with the same bits
    for shares in (1, 2):
        binding.qfc_tune(13, 0)
        binding.qfc_tune(6, 0)
        binding.qfc_tune(14, shares)
        try:
            outs = [torch.full((G, M, d), 9.0, dtype=torch.float16, device=DEV) for _ in range(2)]
            for o in outs:
                binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, o)
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(13, -1)
            binding.qfc_tune(6, -1)
            binding.qfc_tune(14, 0)
        got2 = outs[0].cpu().numpy()
        assert np.all(np.isfinite(got2)), shares
        assert _E(got2.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL, shares
        assert torch.equal(outs[0], outs[1]), shares
    # the launch form of few blocks (walks cut into chunks, partial results combined by a second
    # kernel), forced on: same values within the tolerance, finite, and nothing from past the context
    binding.qfc_tune(6, 1)
    try:
        ws3 = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
        out3 = torch.full((G, M, d), 9.0, dtype=torch.float16, device=DEV)
        binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws3, out3)
        torch.cuda.synchronize()
    finally:
        binding.qfc_tune(6, -1)
    got3 = out3.cpu().numpy()
    assert np.all(np.isfinite(got3))
    assert _E(got3.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL
    # the first token's rows see n_ctx - S + 1 positions only: with one position the output is that value column
    if n_ctx == S:
        assert np.allclose(got[:, :g].astype(np.float64), np.repeat(V[:, None, :, 0], g, axis=1).astype(np.float64), rtol=2e-3, atol=2e-3)


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,n_ctx", [(1, 17, 1, 1, 64, 64, 17), (1, 33, 2, 1, 64, 192, 160), (1, 41, 8, 2, 128, 192, 161),
                                                    (2, 23, 6, 2, 128, 640, 600), (1, 77, 8, 4, 256, 128, 77), (1, 19, 4, 2, 256, 512, 450),
                                                    (1, 150, 10, 2, 128, 192, 150)])
def test_attention_blocks_of_sixteen_query_rows(B, S, h_q, h_kv, d, C, n_ctx):
    """More than 16 query rows in blocks of 16, causal by token: tokens that straddle two blocks, a last block of few
    rows, blocks whose walks end before others', one to eight partial results; against the oracle and
    with what lies past the context poisoned."""
    print(f"attention row blocks B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} n_ctx={n_ctx}", flush=True)
    G, M = B * h_kv, S * (h_q // h_kv)
    rng = np.random.default_rng(n_ctx * 13 + S)
    q = rng.standard_normal((G, M, d)).astype(np.float16)
    K = rng.standard_normal((G, C, d)).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    K[:, 3] = (q[:, 0].astype(np.float32) * 2).astype(np.float16)
    ref = oracle.attention(q, K, V, n_ctx, S)
    K[:, n_ctx:] = np.float16(np.nan)
    V[:, :, n_ctx:] = np.float16(np.inf)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
    qd, kd, vd = torch.from_numpy(q).to(DEV), torch.from_numpy(K).to(DEV), binding.vcache_physical(torch.from_numpy(V).to(DEV))
    for few, splits in ((0, 0), (-1, 0), (1, 0), (1, 1), (1, 3), (1, 8)):
        guard = torch.full((G + 1, M, d), 9.0, dtype=torch.float16, device=DEV)
        binding.qfc_tune(12, splits)
        binding.qfc_tune(13, few)
        try:
            binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, guard[:G])
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(12, 0)
            binding.qfc_tune(13, -1)
        got = guard[:G].cpu().numpy()
        assert np.all(np.isfinite(got)), (few, splits)
        assert _E(got.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL, (few, splits)
        assert bool((guard[G] == 9.0).all())


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,n_ctx", [(1, 17, 1, 1, 64, 64, 33), (1, 64, 2, 1, 128, 64, 64), (1, 129, 3, 1, 64, 192, 161),
                                                    (2, 43, 6, 2, 128, 640, 577), (1, 200, 4, 4, 256, 256, 200), (1, 33, 2, 1, 256, 640, 609),
                                                    (1, 131, 8, 1, 128, 448, 419), (1, 50, 2, 1, 64, 640, 577), (1, 600, 2, 2, 64, 1024, 1000)])
def test_attention_walks_shared_by_wavefronts(B, S, h_q, h_kv, d, C, n_ctx):
    """Prefill with one or two wavefronts per walk, whole walks and walks in chunks: odd numbers of steps (a last stage that lacks
    one), walks of fewer steps than the pipeline has stages and, at each head size, of enough for its branch-free loop, last blocks of few rows; keys that grow along the walk, so
    that the maximum moves in every step; a row of equal scores; everything past the context poisoned."""
    print(f"attention shared walks B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} n_ctx={n_ctx}", flush=True)
    G, M = B * h_kv, S * (h_q // h_kv)
    rng = np.random.default_rng(n_ctx * 29 + S)
    q = rng.standard_normal((G, M, d)).astype(np.float16)
    K = (rng.standard_normal((G, C, d)) * np.linspace(0.2, 1.5, C)[None, :, None]).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    q[:, M // 2] = 0
    ref = oracle.attention(q, K, V, n_ctx, S)
    K[:, n_ctx:] = np.float16(np.nan)
    V[:, :, n_ctx:] = np.float16(np.nan)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
    qd, kd, vd = torch.from_numpy(q).to(DEV), torch.from_numpy(K).to(DEV), binding.vcache_physical(torch.from_numpy(V).to(DEV))
    binding.qfc_tune(13, 0)
    try:
        for shares in (0, 1, 2):
            for chunks in (-1, 0, 2, 3, 8):
                guard = torch.full((G + 1, M, d), 9.0, dtype=torch.float16, device=DEV)
                binding.qfc_tune(14, shares)
                binding.qfc_tune(6, chunks)
                binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, guard[:G])
                torch.cuda.synchronize()
                got = guard[:G].cpu().numpy()
                assert np.all(np.isfinite(got)), (shares, chunks)
                assert _E(got.reshape(G * M, d), ref.reshape(G * M, d)) <= TOL, (shares, chunks)
                assert bool((guard[G] == 9.0).all())
    finally:
        binding.qfc_tune(13, -1)
        binding.qfc_tune(14, 0)
        binding.qfc_tune(6, -1)


@pytest.mark.parametrize("S,h_q,h_kv,d,n_ctx,at", [(20, 2, 1, 64, 155, 135), (17, 6, 2, 128, 21, 4), (9, 4, 1, 256, 90, 81),
                                                   (200, 1, 1, 64, 360, 199), (150, 2, 1, 128, 278, 140), (90, 4, 2, 256, 190, 110),
                                                   (300, 2, 1, 128, 310, 20)])
def test_attention_of_prompts_keeps_infinite_values(S, h_q, h_kv, d, n_ctx, at):
    """Infinite values at position `at`: infinities in those columns of the rows that see it, all other columns as if they were not
    there; walks of odd and even numbers of steps by one or two wavefronts, whole and in chunks, that end at `at` and behind it, at the
    end of the context and before it."""
    print(f"attention infinite values S={S} h_q={h_q} h_kv={h_kv} d={d} n_ctx={n_ctx} at={at}", flush=True)
    g = h_q // h_kv
    C, M = 448, S * g
    rng = np.random.default_rng(n_ctx * 31 + S)
    q = rng.standard_normal((h_kv, M, d)).astype(np.float16)
    K = rng.standard_normal((h_kv, C, d)).astype(np.float16)
    V = rng.standard_normal((h_kv, d, C)).astype(np.float16)
    ref = oracle.attention(q, K, V, n_ctx, S)
    V[:, 3, at], V[:, d - 1, at] = np.float16(np.inf), np.float16(-np.inf)
    seen = max(0, at - (n_ctx - S)) * g  # first row that sees it
    shape = _attn_shape(1, h_q, h_kv, d, C)
    qd, kd, vd = torch.from_numpy(q).to(DEV), torch.from_numpy(K).to(DEV), binding.vcache_physical(torch.from_numpy(V).to(DEV))
    rest = [c for c in range(d) if c not in (3, d - 1)]
    wrong = []
    binding.qfc_tune(13, 0)
    try:
        for shares, chunks in ((1, 0), (2, 0), (1, 2), (2, 2), (1, 3), (2, 3), (2, 8)):
            binding.qfc_tune(14, shares)
            binding.qfc_tune(6, chunks)
            ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
            out = torch.empty((h_kv, M, d), dtype=torch.float16, device=DEV)
            binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, out)
            got = out.cpu().numpy()
            if not (np.all(got[:, seen:, 3] == np.inf) and np.all(got[:, seen:, d - 1] == -np.inf) and np.all(np.isfinite(got[..., rest])) and
                    _E(got[..., rest].reshape(h_kv * M, d - 2), ref[..., rest].reshape(h_kv * M, d - 2)) <= TOL):
                wrong.append((shares, chunks))
    finally:
        binding.qfc_tune(13, -1)
        binding.qfc_tune(14, 0)
        binding.qfc_tune(6, -1)
    assert wrong == []


@pytest.mark.parametrize("B,S,h_q,h_kv,d,n_ctx", [(1, 1, 8, 2, 64, 400), (2, 1, 32, 8, 128, 290), (1, 2, 4, 1, 256, 448), (1, 20, 4, 2, 128, 411)])
def test_attention_of_few_rows_keeps_infinite_values(B, S, h_q, h_kv, d, n_ctx):
    """The same at the first position of the last token and at position 0 for walks split over workgroups: any number of partial
    results, of which the combination takes eight at a time."""
    print(f"attention infinite values, few rows B={B} S={S} h_q={h_q} h_kv={h_kv} d={d} n_ctx={n_ctx}", flush=True)
    C, G, M = 448, B * h_kv, S * (h_q // h_kv)
    rng = np.random.default_rng(n_ctx * 37 + S)
    q = rng.standard_normal((G, M, d)).astype(np.float16)
    K = rng.standard_normal((G, C, d)).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    ref = oracle.attention(q, K, V, n_ctx, S)
    V[:, 3, n_ctx - S], V[:, d - 1, 0] = np.float16(np.inf), np.float16(-np.inf)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    qd, kd, vd = torch.from_numpy(q).to(DEV), torch.from_numpy(K).to(DEV), binding.vcache_physical(torch.from_numpy(V).to(DEV))
    rest = [c for c in range(d) if c not in (3, d - 1)]
    wrong = []
    try:
        for splits in (0, 1, 2, 3, 7):
            binding.qfc_tune(12, splits)
            binding.qfc_tune(13, 1)
            ws = torch.empty(binding.qfc_attention_workspace_size(shape, S), dtype=torch.uint8, device=DEV)
            out = torch.empty((G, M, d), dtype=torch.float16, device=DEV)
            binding.qfc_attention(qd, kd, vd, S, n_ctx, shape, ws, out)
            got = out.cpu().numpy()
            if not (np.all(got[..., 3] == np.inf) and np.all(got[..., d - 1] == -np.inf) and np.all(np.isfinite(got[..., rest])) and
                    _E(got[..., rest].reshape(G * M, d - 2), ref[..., rest].reshape(G * M, d - 2)) <= TOL):
                wrong.append(splits)
    finally:
        binding.qfc_tune(12, 0)
        binding.qfc_tune(13, -1)
    assert wrong == []


def test_attention_few_blocks_needs_the_larger_workspace():
    """Few blocks of query rows (fewer than compute units): the walks may be cut into chunks, whose
    partial results live in the workspace; the size query says how much, a smaller one is refused."""
    B, S, h_q, h_kv, d, C = 1, 640, 8, 4, 256, 640
    shape = _attn_shape(B, h_q, h_kv, d, C)
    need = binding.qfc_attention_workspace_size(shape, S)
    G, M = B * h_kv, S * (h_q // h_kv)
    assert need == G * M * 8 * (d + 2) * 4
    q = torch.zeros((G, M, d), dtype=torch.float16, device=DEV)
    kc = torch.zeros((G, C, d), dtype=torch.float16, device=DEV)
    vc = torch.zeros((G, C // 64, d, 64), dtype=torch.float16, device=DEV)
    out = torch.empty_like(q)
    ws = torch.empty(need - 16, dtype=torch.uint8, device=DEV)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_attention(q, kc, vc, S, S, shape, ws, out)
    assert e.value.code == binding.QFC_ERR_BUFFER_TOO_SMALL
    # many blocks: no partial results, the minimum suffices
    big = _attn_shape(1, 32, 8, 128, 4096)
    assert binding.qfc_attention_workspace_size(big, 4096) == 256


def test_rope_then_attention_decode_step():
    """One decode step end to end: the token's QKV row goes through the rotary kernel into the caches
    and attention reads them; compared with the oracle's pipeline on the same binary16 caches."""
    B, h_q, h_kv, d, C, pos0 = 2, 8, 2, 128, 256, 100
    G, g = B * h_kv, h_q // h_kv
    rng = np.random.default_rng(12)
    K = rng.standard_normal((G, C, d)).astype(np.float16)
    V = rng.standard_normal((G, d, C)).astype(np.float16)
    qkv = synth.activations(3900, 0, 0, B, (h_q + 2 * h_kv) * d).reshape(B, 1, -1)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    q_out = torch.empty((G, g, d), dtype=torch.float16, device=DEV)
    kc, vc = torch.from_numpy(K).to(DEV), binding.vcache_physical(torch.from_numpy(V).to(DEV))
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, 1), dtype=torch.uint8, device=DEV)
    out = torch.empty((G, g, d), dtype=torch.float16, device=DEV)
    binding.qfc_rope_qkv(torch.from_numpy(qkv).to(DEV), pos0, shape, 10000.0, q_out, kc, vc)
    binding.qfc_attention(q_out, kc, vc, 1, pos0 + 1, shape, ws, out)
    torch.cuda.synchronize()
    q_ref, k_ref, v_ref = oracle.rope_qkv_layout(qkv, pos0, h_q, h_kv, d, 10000.0)
    K[:, pos0] = k_ref[:, 0]
    V[:, :, pos0] = v_ref[:, 0]
    ref = oracle.attention(q_ref, K, V, pos0 + 1, 1)
    assert _E(out.cpu().numpy().reshape(G * g, d), ref.reshape(G * g, d)) <= TOL
    # [G, g, d] is [B, h_q * d]: query head kv * g + j of batch b at row b, columns (kv * g + j) * d ..
    assert out.reshape(B, h_q * d).shape == (B, h_q * d)


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("B,h_q,h_kv,d,C,pos0,K,norm", [(1, 4, 2, 64, 64, 0, 128, False), (2, 8, 2, 128, 128, 77, 1152, True),
                                                         (1, 32, 8, 128, 8192, 8191, 4096, True), (8, 8, 4, 256, 192, 130, 2304, False),
                                                         (3, 2, 1, 128, 131072, 131071, 256, False)])
def test_qkv_layer_with_rotary_embedding_merged(fmt, B, h_q, h_kv, d, C, pos0, K, norm):
    """QKV layer + rotary embedding + layout transformation + cache append in one decode launch against
    the oracle's pipeline on the unrounded projection outputs, and against the two-launch route."""
    print(f"qkv+rope {fmt} B={B} h_q={h_q} h_kv={h_kv} d={d} C={C} pos0={pos0} K={K} norm={norm}", flush=True)
    base = 500000.0 if d == 128 else 10000.0
    N = (h_q + 2 * h_kv) * d
    G, g = B * h_kv, h_q // h_kv
    fc = synth.FC("qkv", K, N, fmt)
    wq, s = synth.weights(3950, B, d, fc)
    x = synth.activations(3950, B, d, B, K)
    gamma = (1.0 + 0.1 * synth.activations(3951, B, d, 1, K)[0].astype(np.float32)).astype(np.float16)
    layer = _layer(wq, s, fmt)
    shape = _attn_shape(B, h_q, h_kv, d, C)
    table = binding.qfc_rope_table(shape, base, pos0 + 1)
    # the table is the fp64 cosine and sine, rounded to binary32
    i = np.arange(d // 2, dtype=np.float64)
    ang = float(pos0) * base ** (-2.0 * i / d)
    t = table.cpu().numpy()
    assert np.allclose(t[pos0, :, 0], np.cos(ang), rtol=0, atol=2.0 ** -23) and np.allclose(t[pos0, :, 1], np.sin(ang), rtol=0, atol=2.0 ** -23)
    assert np.array_equal(t[0, :, 0], np.ones(d // 2, dtype=np.float32)) and not t[0, :, 1].any()
    xd = torch.from_numpy(x).to(DEV)
    gd = torch.from_numpy(gamma).to(DEV)
    q_out = torch.zeros((G, g, d), dtype=torch.float16, device=DEV)
    kc = torch.full((G, C, d), 3.0, dtype=torch.float16, device=DEV)
    vc = torch.full((G, C // 64, d, 64), 5.0, dtype=torch.float16, device=DEV)
    kw = dict(norm_gamma=gd, norm_eps=1e-5) if norm else {}
    binding.qfc_forward_qkv_rope(layer.handle, xd, pos0, shape, table, q_out, kc, vc, **kw)
    torch.cuda.synchronize()
    # oracle: the real projection (with the merged normalization in its factorised form, as for the
    # plain layer: rs * fc(fp16(x * weight))), then the real rotation; one rounding at the end
    if norm:
        y_ref = oracle.rms_scale(x, 1e-5)[:, None] * oracle.fc_weight_only(oracle.norm_weighted_input(x, gamma, 0.0), wq, s, _group(fmt))
    else:
        y_ref = oracle.fc_weight_only(x, wq, s, _group(fmt))
    q_ref, k_ref, v_ref = oracle.rope_qkv_layout_exact(y_ref.reshape(B, 1, N), pos0, h_q, h_kv, d, base)
    kcn, vcn = kc.cpu().numpy(), binding.vcache_logical(vc).cpu().numpy()
    got = np.concatenate([q_out.cpu().numpy().reshape(B, h_kv, g * d), kcn[:, pos0].reshape(B, h_kv, d),
                          vcn[:, :, pos0].reshape(B, h_kv, d)], axis=2).reshape(B, -1)
    ref = np.concatenate([q_ref.reshape(B, h_kv, g * d), k_ref.reshape(B, h_kv, d), v_ref.reshape(B, h_kv, d)], axis=2).reshape(B, -1)
    assert _E(got, ref) <= TOL
    # nothing but position pos0 of the caches changed
    kcn[:, pos0] = 3.0
    vcn[:, :, pos0] = 5.0
    assert np.all(kcn == 3.0) and np.all(vcn == 5.0)
    # the two-launch route (layer, then the rotary kernel) rounds the projection to binary16 in between
    y = torch.empty((B, N), dtype=torch.float16, device=DEV)
    if norm:
        binding.qfc_forward_fused(layer.handle, xd, y, norm_gamma=gd, norm_eps=1e-5)
    else:
        binding.qfc_forward(layer.handle, xd, y)
    q2 = torch.zeros_like(q_out)
    kc2 = torch.full_like(kc, 3.0)
    vc2 = torch.full_like(vc, 5.0)
    binding.qfc_rope_qkv(y.view(B, 1, N), pos0, shape, base, q2, kc2, vc2)
    torch.cuda.synchronize()
    got2 = np.concatenate([q2.cpu().numpy().reshape(B, h_kv, g * d), kc2.cpu().numpy()[:, pos0].reshape(B, h_kv, d),
                           binding.vcache_logical(vc2).cpu().numpy()[:, :, pos0].reshape(B, h_kv, d)], axis=2).reshape(B, -1)
    assert _E(got, got2.astype(np.float64)) <= 2 * TOL
    # values are not rotated: the same sums, the same single rounding, the same bits
    assert np.array_equal(binding.vcache_logical(vc).cpu().numpy()[:, :, pos0].view(np.uint16),
                          binding.vcache_logical(vc2).cpu().numpy()[:, :, pos0].view(np.uint16))
    layer.close()


def test_qkv_layer_with_rotary_embedding_rejects_what_it_cannot_do():
    B, h_q, h_kv, d, C = 1, 4, 2, 64, 64
    N, K = (h_q + 2 * h_kv) * d, 128
    fc = synth.FC("qkv", K, N, "w8c")
    wq, s = synth.weights(3960, 0, 0, fc)
    layer = _layer(wq, s, "w8c")
    shape = _attn_shape(B, h_q, h_kv, d, C)
    table = binding.qfc_rope_table(shape, 10000.0, 8)
    x = torch.zeros((B, K), dtype=torch.float16, device=DEV)
    q = torch.zeros((B * h_kv, h_q // h_kv, d), dtype=torch.float16, device=DEV)
    kc = torch.zeros((B * h_kv, C, d), dtype=torch.float16, device=DEV)
    vc = torch.zeros((B * h_kv, C // 64, d, 64), dtype=torch.float16, device=DEV)
    for pos in (-1, 8, 64):  # before the cache, beyond the table, beyond the cache
        with pytest.raises(binding.QfcError) as e:
            binding.qfc_forward_qkv_rope(layer.handle, x, pos, shape, table, q, kc, vc)
        assert e.value.code == binding.QFC_ERR_INVALID_ARG
    wrong = _attn_shape(B, h_q + 2, h_kv, d, C)  # N does not match the shape
    with pytest.raises((binding.QfcError, ValueError)):
        binding.qfc_forward_qkv_rope(layer.handle, x, 0, wrong, table,
                                     torch.zeros((B * h_kv, (h_q + 2) // h_kv, d), dtype=torch.float16, device=DEV), kc, vc)
    layer.close()
    l8 = _layer(wq, s, "w8c", mode=binding.QFC_COMPUTE_INT8_ACT_DECODE)
    with pytest.raises(binding.QfcError) as e:
        binding.qfc_forward_qkv_rope(l8.handle, x, 0, shape, table, q, kc, vc)
    assert e.value.code == binding.QFC_ERR_UNSUPPORTED
    l8.close()


# ------------------------------------------------------------------ one decoder layer, decode step, every operator chained
def test_decoder_layer_decode_step_chain():
    """rmsnorm -> QKV layer -> rotary + layouts + cache append -> attention -> O layer + residual ->
    rmsnorm -> gate+up layer with gated output -> down layer + residual, M = B token rows.
    Every stage is compared with the oracle applied to the tensors the previous GPU stage stored
    (so each comparison carries one stage's error), and the layouts line up without any glue."""
    B, hidden, h_q, h_kv, d, ffn, C, pos0 = 2, 512, 8, 2, 64, 1024, 128, 77
    G, g = B * h_kv, h_q // h_kv
    eps = 1e-5
    rng = np.random.default_rng(41)

    def mk(name, K, N, fmt, seed):
        fc = synth.FC(name, K, N, fmt)
        wq, s = synth.weights(4000, seed, 0, fc)
        if fmt == "w4g32":
            s = (s.astype(np.float32) * 0.25).astype(np.float16)  # keep the chain's magnitudes moderate
        else:
            s = (s * 0.05).astype(np.float32)
        return wq, s, _layer(wq, s, fmt)

    wq_qkv, s_qkv, l_qkv = mk("qkv", hidden, (h_q + 2 * h_kv) * d, "w4g32", 1)
    wq_o, s_o, l_o = mk("o", h_q * d, hidden, "w4g32", 2)
    wq_gu, s_gu, l_gu = mk("gate_up", hidden, 2 * ffn, "w4g32", 3)
    wq_dn, s_dn, l_dn = mk("down", ffn, hidden, "w4g32", 4)
    h0 = synth.activations(4000, 0, 9, B, hidden)
    g1 = (1 + 0.1 * rng.standard_normal(hidden)).astype(np.float16)
    g2 = (1 + 0.1 * rng.standard_normal(hidden)).astype(np.float16)
    K0 = rng.standard_normal((G, C, d)).astype(np.float16)
    V0 = rng.standard_normal((G, d, C)).astype(np.float16)
    shape = _attn_shape(B, h_q, h_kv, d, C)

    T = lambda a: torch.from_numpy(a).to(DEV)
    E = lambda *sh: torch.empty(sh, dtype=torch.float16, device=DEV)
    h_d, g1_d, g2_d = T(h0), T(g1), T(g2)
    kc, vc = T(K0), binding.vcache_physical(T(V0))
    x1, qkv, q, att, h1, x2, a, h2 = E(B, hidden), E(B, 1, (h_q + 2 * h_kv) * d), E(G, g, d), E(G, g, d), E(B, hidden), E(B, hidden), E(B, ffn), E(B, hidden)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, 1), dtype=torch.uint8, device=DEV)

    binding.qfc_rmsnorm(h_d, g1_d, eps, 0.0, y=x1)
    binding.qfc_forward(l_qkv.handle, x1, qkv.view(B, -1))
    binding.qfc_rope_qkv(qkv, pos0, shape, 10000.0, q, kc, vc)
    binding.qfc_attention(q, kc, vc, 1, pos0 + 1, shape, ws, att)
    binding.qfc_forward_fused(l_o.handle, att.view(B, h_q * d), h1, residual=h_d)
    binding.qfc_rmsnorm(h1, g2_d, eps, 0.0, y=x2)
    binding.qfc_forward_fused(l_gu.handle, x2, a, activation=binding.QFC_ACT_SILU, gated_output=True)
    binding.qfc_forward_fused(l_dn.handle, a, h2, residual=h1)
    torch.cuda.synchronize()
    N = lambda t: t.cpu().numpy()
    err = oracle.floored_rel_error

    _, x1_ref = oracle.rmsnorm(h0, g1, eps)
    assert err(N(x1), x1_ref) <= TOL
    assert err(N(qkv).reshape(B, -1), oracle.fc_weight_only(N(x1), wq_qkv, s_qkv, 32)) <= TOL
    q_ref, k_ref, v_ref = oracle.rope_qkv_layout(N(qkv), pos0, h_q, h_kv, d, 10000.0)
    assert err(N(q).reshape(G * g, d), q_ref.reshape(G * g, d).astype(np.float64)) <= TOL
    K1, V1 = K0.copy(), V0.copy()
    K1[:, pos0], V1[:, :, pos0] = N(kc)[:, pos0], N(binding.vcache_logical(vc))[:, :, pos0]
    assert err(K1[:, pos0], k_ref[:, 0].astype(np.float64)) <= TOL and np.array_equal(V1[:, :, pos0], v_ref[:, 0])
    att_ref = oracle.attention(N(q), K1, V1, pos0 + 1, 1)
    assert err(N(att).reshape(G * g, d), att_ref.reshape(G * g, d)) <= TOL
    # the attention output [G, g, d] is [B, h_q * d] as it stands: head kv * g + j of batch b
    o_ref = oracle.add_residual(oracle.fc_weight_only(N(att).reshape(B, h_q * d), wq_o, s_o, 32), h0)
    assert err(N(h1), o_ref) <= TOL
    _, x2_ref = oracle.rmsnorm(N(h1), g2, eps)
    assert err(N(x2), x2_ref) <= TOL
    a_ref = oracle.gated_output(oracle.fc_weight_only(N(x2), wq_gu, s_gu, 32), oracle.SILU)
    assert err(N(a), a_ref) <= TOL
    h2_ref = oracle.add_residual(oracle.fc_weight_only(N(a), wq_dn, s_dn, 32), N(h1))
    assert err(N(h2), h2_ref) <= TOL
    assert np.all(np.isfinite(N(h2)))

    # The same layer in six launches: both normalizations merged into the layers that follow them, the
    # rotary kernel merged into the QKV layer.  Fewer roundings on the way, so the end of the layer
    # is compared with the eight-launch result (each differs from the real chain by its own roundings).
    table = binding.qfc_rope_table(shape, 10000.0, pos0 + 1)
    kc6, vc6 = T(K0), binding.vcache_physical(T(V0))
    q6, att6, h16, a6, h26 = E(G, g, d), E(G, g, d), E(B, hidden), E(B, ffn), E(B, hidden)
    binding.qfc_forward_qkv_rope(l_qkv.handle, h_d, pos0, shape, table, q6, kc6, vc6, norm_gamma=g1_d, norm_eps=eps)
    binding.qfc_attention(q6, kc6, vc6, 1, pos0 + 1, shape, ws, att6)
    binding.qfc_forward_fused(l_o.handle, att6.view(B, h_q * d), h16, residual=h_d)
    binding.qfc_forward_fused(l_gu.handle, h16, a6, activation=binding.QFC_ACT_SILU, gated_output=True, norm_gamma=g2_d, norm_eps=eps)
    binding.qfc_forward_fused(l_dn.handle, a6, h26, residual=h16)
    torch.cuda.synchronize()
    assert err(N(q6).reshape(G * g, d), N(q).reshape(G * g, d).astype(np.float64)) <= 2 * TOL
    assert err(N(kc6)[:, pos0], N(kc)[:, pos0].astype(np.float64)) <= 2 * TOL
    assert err(N(att6).reshape(G * g, d), N(att).reshape(G * g, d).astype(np.float64)) <= 2 * TOL
    assert err(N(h26), N(h2).astype(np.float64)) <= 4 * TOL  # (five stages, each within its own bound of the real chain)
    for l in (l_qkv, l_o, l_gu, l_dn):
        l.close()


@pytest.mark.parametrize("fmt", ["w8c", "w4g32", "w4c"])
@pytest.mark.parametrize("N,K", [(32, 96), (130, 256), (1000, 2304), (96, 14336)])
def test_decode_norm_merged_into_layer(fmt, N, K):
    """RMS normalization merged into the decode kernel: y = rs * fc(fp16(x * weight)) (+ residual),
    also together with the gated output (the gate+up layer of a decoder layer)."""
    fc = synth.FC("t", K, N, fmt)
    wq, s = synth.weights(3950, N, K, fc)
    layer = _layer(wq, s, fmt)
    gamma = (synth.activations(3951, N, K, 1, K)[0] * np.float16(0.5)).astype(np.float16)
    gd = torch.from_numpy(gamma).to(DEV)
    for M in (1, 2, 4, 5, 8):
        print(f"decode norm merged {fmt} N={N} K={K} M={M}", flush=True)
        x = synth.activations(3950, N, K + M, M, K)
        res = synth.activations(3952, N, K + M, M, N)
        off, eps = (1.0, 1e-6) if M % 2 else (0.0, 1e-5)
        xd, rd = torch.from_numpy(x).to(DEV), torch.from_numpy(res).to(DEV)
        y = torch.empty((M, N), dtype=torch.float16, device=DEV)
        binding.qfc_forward_fused(layer.handle, xd, y, residual=rd, norm_gamma=gd, norm_eps=eps, norm_offset=off)
        torch.cuda.synchronize()
        x_in = oracle.norm_weighted_input(x, gamma, off)
        rs = oracle.rms_scale(x, eps)
        full = rs[:, None] * oracle.fc_weight_only(x_in, wq, s, _group(fmt))
        assert _E(y.cpu().numpy(), oracle.add_residual(full, res)) <= TOL, M
        # ... and against the plain definition: the layer applied to rmsnorm(x), nothing factored
        # out and nothing rounded between the normalization and the product.  The merged operator
        # rounds the layer's input once to binary16 (FP16 activations; an unfused normalization
        # would store the same precision), which the plain definition does not: K independent
        # roundings of relative size <= 2^-11 add an error of standard deviation
        # sigma[m,n] <= 2^-11 / sqrt(3) * sqrt(sum_k (xn[m,k] W[n,k])^2) to output (m,n); six of them
        # are allowed on top of the bound of the output rounding.
        xn, What = oracle.rmsnorm(x, gamma, eps, off)[1], oracle.dequantize(wq, s, _group(fmt))
        plain = oracle.add_residual(xn @ What.T, res)
        sigma = 2.0 ** -11 / np.sqrt(3.0) * np.sqrt((xn * xn) @ (What * What).T)
        dev = np.abs(y.cpu().numpy().astype(np.float64) - plain)
        assert np.all(dev <= TOL * oracle.floored_denominator(plain) + 6.0 * sigma), M
        assert _E(y.cpu().numpy(), plain) <= 1.5 * TOL, M  # (and never far from the plain bound)
        if N % 32 == 0:
            yg = torch.empty((M, N // 2), dtype=torch.float16, device=DEV)
            # a normalization weight scaled down (by a power of two) keeps the product of the two halves of order 1..64
            # (the input's own scale cancels in the normalization)
            mag = np.max(np.abs(rs[:, None] * oracle.fc_weight_only(oracle.norm_weighted_input(x, gamma, 0.0), wq, s, _group(fmt))))
            shrink = 2.0 ** min(0, int(np.floor(np.log2(8.0 / mag))))
            gs = (gamma.astype(np.float32) * shrink).astype(np.float16)
            xs = x
            binding.qfc_forward_fused(layer.handle, torch.from_numpy(xs).to(DEV), yg, activation=binding.QFC_ACT_SILU,
                                      gated_output=True, norm_gamma=torch.from_numpy(gs).to(DEV), norm_eps=eps,
                                      norm_offset=0.0)
            torch.cuda.synchronize()
            fulls = oracle.rms_scale(xs, eps)[:, None] * oracle.fc_weight_only(oracle.norm_weighted_input(xs, gs, 0.0), wq, s, _group(fmt))
            assert _E(yg.cpu().numpy(), oracle.gated_output(fulls, oracle.SILU)) <= TOL, M
            plains = oracle.rmsnorm(xs, gs, eps, 0.0)[1] @ oracle.dequantize(wq, s, _group(fmt)).T
            assert _E(yg.cpu().numpy(), oracle.gated_output(plains, oracle.SILU)) <= 2 * TOL, M  # (two rounded-input sums multiplied)
    # against the unfused sequence on the GPU: norm kernel, then the plain layer
    x = synth.activations(3953, N, K, 3, K)
    xd = torch.from_numpy(x).to(DEV)
    yn = torch.empty((3, K), dtype=torch.float16, device=DEV)
    y_a = torch.empty((3, N), dtype=torch.float16, device=DEV)
    y_b = torch.empty((3, N), dtype=torch.float16, device=DEV)
    if K <= 14336:
        binding.qfc_rmsnorm(xd, gd, 1e-5, 0.0, y=yn)
        binding.qfc_forward(layer.handle, yn, y_a)
        binding.qfc_forward_fused(layer.handle, xd, y_b, norm_gamma=gd, norm_eps=1e-5, norm_offset=0.0)
        torch.cuda.synchronize()
        assert _E(y_b.cpu().numpy(), y_a.cpu().numpy().astype(np.float64)) <= 2 * TOL
    layer.close()


def test_probe_mfma_runs_and_rejects_bad_arguments():
    """The measurement probe of qfc_experimental.h: a short run writes both counters of every
    workgroup; arguments outside its documented ranges are refused before any launch."""
    print("mfma probe", flush=True)
    for kind, operands in ((0, True), (1, True), (4, 0), (4, 1), (4, 2), (4, 3), (5, 0), (5, 1), (5, 2), (5, 3)):
        ticks = torch.zeros((8, 2), dtype=torch.int64, device=DEV)
        binding.qfc_probe_mfma(kind, operands, 10, 8, ticks)
        torch.cuda.synchronize()
        t = ticks.cpu().numpy()
        assert (t > 0).all()
    ticks = torch.zeros((8, 2), dtype=torch.int64, device=DEV)
    for args in ((2, True, 10, 8), (0, True, 0, 8), (0, True, (1 << 22) + 1, 8)):
        with pytest.raises(binding.QfcError):
            binding.qfc_probe_mfma(*args, ticks)
    with pytest.raises(ValueError):
        binding.qfc_probe_mfma(0, True, 10, 4097, ticks)


@pytest.mark.parametrize("fmt,mode", [("w4g32", None), ("w4c", None), ("w8c", binding.QFC_COMPUTE_FP16_DEQUANT),
                                      ("w8c", None), ("w4c", binding.QFC_COMPUTE_INT8_ACT)])
@pytest.mark.parametrize("M,N,K,row_tiles", [(9, 1, 32, 0), (16, 50, 160, 1), (17, 100, 96, 3), (33, 130, 416, 2),
                                             (32, 1000, 1184, 7), (48, 264, 2304, 5), (64, 96, 14336, 4), (63, 300, 544, 0)])
def test_few_token_rows_match_oracle(fmt, mode, M, N, K, row_tiles):
    """The kernels for 9 to 64 token rows at the edges of their blocks of 8 and 16 rows, with K ending inside a step,
    fewer steps than wavefronts, a last workgroup that is not full, and a residual."""
    print(f"few token rows {fmt} mode={mode} M={M} N={N} K={K} row tiles={row_tiles}", flush=True)
    wq, s = synth.weights(6000, M, N, synth.FC("t", K, N, fmt))
    x = synth.activations(6000, M, N, M, K)
    res = synth.activations(6000, M, N + 1, M, N)
    layer = _layer(wq, s, fmt, max_m=M, mode=mode)
    int8 = mode == binding.QFC_COMPUTE_INT8_ACT or (fmt == "w8c" and mode is None)
    ref = oracle.fc_int8_act(x, wq, s)[3] if int8 else oracle.fc_weight_only(x, wq, s, _group(fmt))
    xd, rd = torch.from_numpy(x).to(DEV), torch.from_numpy(res).to(DEV)
    guard = torch.full((M + 1, N), 77.0, dtype=torch.float16, device=DEV)  # the row behind y stays as it is
    y = guard[:M]
    binding.qfc_tune(8, row_tiles)
    try:
        binding.qfc_forward(layer.handle, xd, y)
        plain = y.cpu().numpy()
        binding.qfc_forward_fused(layer.handle, xd, y, residual=rd)
        torch.cuda.synchronize()
    finally:
        binding.qfc_tune(8, 0)
    assert _E(plain, ref) <= TOL
    assert _E(y.cpu().numpy(), ref + res.astype(np.float64)) <= TOL
    assert bool((guard[M] == 77.0).all())
    if int8:  # exact sums and the same rounding steps: the same bits as the large kernel
        binding.qfc_tune(9, 0)
        try:
            big = _forward(layer, x)
        finally:
            binding.qfc_tune(9, -1)
        assert np.array_equal(plain.view(np.uint16), big.view(np.uint16))
    layer.close()


def _with_infinities(x, wq, ref):
    """Puts an infinity into three rows of x (first octets, last element of K) and what the definition gives for it
    (NaN where its weight is zero) into the same rows of ref; returns the rows that stay finite."""
    M, K = x.shape
    for row, k, sign in ((0, 3, 1.0), (M // 2, K - 1, -1.0), (M - 1, 31, 1.0)):
        x[row, k] = np.float16(sign * np.inf)
        w = np.asarray(wq)[:, k]
        ref[row] = np.where(w == 0, np.nan, np.where((w > 0) == (sign > 0), np.inf, -np.inf))
    return np.isfinite(ref).all(axis=1)


@pytest.mark.parametrize("fmt", ["w4g32", "w4c", "w8c"])
@pytest.mark.parametrize("K", [160, 4640, 5088])
def test_decode_infinite_activations(fmt, K):
    """An infinite activation gives its row the infinity the definition gives and leaves the other rows alone, wherever K ends in
    a step of 128: staged through registers and by direct copies (five token rows and more, long K, 4-bit weights)."""
    N = 90
    for M in (4, 5, 8):
        print(f"infinite activations, decode {fmt} M={M} K={K}", flush=True)
        wq, s = synth.weights(6051, M, K, synth.FC("t", K, N, fmt))
        x = synth.activations(6051, M, K, M, K)
        ref = oracle.fc_weight_only(x, wq, s, _group(fmt))
        finite = _with_infinities(x, wq, ref)
        layer = _layer(wq, s, fmt, max_m=M, mode=binding.QFC_COMPUTE_FP16_DEQUANT)
        y = _forward(layer, x).astype(np.float64)
        assert finite.sum() == M - 3
        assert _E(y[finite], ref[finite]) <= TOL, M
        assert np.array_equal(y[~finite], ref[~finite], equal_nan=True), M
        layer.close()


@pytest.mark.parametrize("fmt", ["w4g32", "w4c", "w8c"])
@pytest.mark.parametrize("M,K", [(9, 160), (24, 64), (33, 352), (64, 544), (100, 160), (100, 224)])
def test_few_token_rows_infinite_activations(fmt, M, K):
    """An infinite activation gives its row the infinity the definition gives (NaN where its weight is zero), wherever
    K ends in a step of 128, and leaves the other rows alone: also in the large kernels at the same sizes."""
    print(f"infinite activations {fmt} M={M} K={K}", flush=True)
    N = 90
    wq, s = synth.weights(6050, M, K, synth.FC("t", K, N, fmt))
    x = synth.activations(6050, M, K, M, K)
    ref = oracle.fc_weight_only(x, wq, s, _group(fmt))
    finite = _with_infinities(x, wq, ref)
    assert finite.sum() == M - 3
    layer = _layer(wq, s, fmt, max_m=M, mode=binding.QFC_COMPUTE_FP16_DEQUANT)
    for max_m in (1024, 0):  # the kernels for few token rows, the large ones
        binding.qfc_tune(9, max_m)
        try:
            y = _forward(layer, x).astype(np.float64)
        finally:
            binding.qfc_tune(9, -1)
        assert _E(y[finite], ref[finite]) <= TOL, max_m
        assert np.array_equal(y[~finite], ref[~finite], equal_nan=True), max_m
    layer.close()


@pytest.mark.parametrize("fmt,mode", [("w4g32", None), ("w4c", None), ("w8c", binding.QFC_COMPUTE_FP16_DEQUANT),
                                      ("w8c", None), ("w4c", binding.QFC_COMPUTE_INT8_ACT)])
@pytest.mark.parametrize("M,N,K,row_tiles,blocks", [(65, 40, 160, 0, 0), (77, 300, 2304, 2, 0), (96, 130, 416, 3, 0), (97, 130, 416, 4, 0),
                                                    (129, 1000, 96, 1, 0), (250, 70, 544, 0, 6), (300, 264, 1184, 3, 0), (513, 96, 2048, 0, 0), (100, 200, 256, 8, 4)])
def test_blocks_of_token_rows_match_oracle(fmt, mode, M, N, K, row_tiles, blocks):
    """More than 64 token rows in blocks of equal size: blocks that end past the last row, a last block of few rows,
    row groups that do not fill all XCDs; and the tiles of the large kernels at the same sizes."""
    print(f"blocks of token rows {fmt} mode={mode} M={M} N={N} K={K} row tiles={row_tiles} blocks={blocks}", flush=True)
    wq, s = synth.weights(6100, M, N, synth.FC("t", K, N, fmt))
    x = synth.activations(6100, M, N, M, K)
    res = synth.activations(6100, M, N + 1, M, N)
    layer = _layer(wq, s, fmt, max_m=M, mode=mode)
    int8 = mode == binding.QFC_COMPUTE_INT8_ACT or (fmt == "w8c" and mode is None)
    ref = oracle.fc_int8_act(x, wq, s)[3] if int8 else oracle.fc_weight_only(x, wq, s, _group(fmt))
    xd, rd = torch.from_numpy(x).to(DEV), torch.from_numpy(res).to(DEV)
    outs = []
    for max_m in (1024, 0):  # these kernels, the large ones
        guard = torch.full((M + 1, N), 77.0, dtype=torch.float16, device=DEV)
        y = guard[:M]
        binding.qfc_tune(8, row_tiles)
        binding.qfc_tune(9, max_m)
        binding.qfc_tune(11, blocks)
        try:
            binding.qfc_forward(layer.handle, xd, y)
            outs.append(y.cpu().numpy())
            binding.qfc_forward_fused(layer.handle, xd, y, residual=rd)
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(8, 0)
            binding.qfc_tune(9, -1)
            binding.qfc_tune(11, 0)
        assert _E(outs[-1], ref) <= TOL, max_m
        assert _E(y.cpu().numpy(), ref + res.astype(np.float64)) <= TOL, max_m
        assert bool((guard[M] == 77.0).all())
    if int8:
        assert np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))
    layer.close()


@pytest.mark.parametrize("fmt,mode", [("w4g32", None), ("w4c", None), ("w8c", binding.QFC_COMPUTE_FP16_DEQUANT),
                                      ("w8c", None), ("w4c", binding.QFC_COMPUTE_INT8_ACT)])
@pytest.mark.parametrize("N,K", [(645, 4128), (2304, 1024), (2100, 4096)])
def test_narrow_layers_in_more_blocks_than_needed(fmt, mode, N, K):
    """Layers of few row tiles, whose token rows the library cuts into blocks of 16 to 48 by itself: numbers of rows whose last
    block is one row, nearly full or full.  (K = 4096: with int4 codes and int8 activations workgroups begin at different k.)"""
    wq, s = synth.weights(6400, N, K, synth.FC("t", K, N, fmt))
    layer = _layer(wq, s, fmt, max_m=144, mode=mode)
    int8 = mode == binding.QFC_COMPUTE_INT8_ACT or (fmt == "w8c" and mode is None)
    for M in (17, 31, 33, 48, 64, 65, 97, 144):
        print(f"narrow layer {fmt} mode={mode} N={N} K={K} M={M}", flush=True)
        x = synth.activations(6400, M, N, M, K)
        guard = torch.full((M + 1, N), 77.0, dtype=torch.float16, device=DEV)
        binding.qfc_forward(layer.handle, torch.from_numpy(x).to(DEV), guard[:M])
        y = guard[:M].cpu().numpy()
        if int8:
            assert _E(y, oracle.fc_int8_act(x, wq, s)[3]) <= TOL, M
            binding.qfc_tune(9, 0)
            try:
                large = _forward(layer, x)
            finally:
                binding.qfc_tune(9, -1)
            assert np.array_equal(y.view(np.uint16), np.asarray(large).view(np.uint16)), M
        else:
            assert _E(y, oracle.fc_weight_only(x, wq, s, _group(fmt))) <= TOL, M
        assert bool((guard[M] == 77.0).all()), M
    layer.close()


@pytest.mark.parametrize("fmt,mode", [("w4g32", None), ("w4c", None), ("w8c", binding.QFC_COMPUTE_FP16_DEQUANT),
                                      ("w8c", None), ("w4c", binding.QFC_COMPUTE_INT8_ACT)])
@pytest.mark.parametrize("N,K", [(32512, 128), (32768, 160), (49152, 128), (65792, 96)])
def test_wide_layers_of_few_token_rows(fmt, mode, N, K):
    """On both sides of the lines (numbers of rows and channels) between the kernels for few token rows and the tiles
    that fill half the chip and more: either kernel's result."""
    print(f"wide layer {fmt} mode={mode} N={N} K={K}", flush=True)
    wq, s = synth.weights(6300, N, K, synth.FC("t", K, N, fmt))
    layer = _layer(wq, s, fmt, max_m=64, mode=mode)
    int8 = mode == binding.QFC_COMPUTE_INT8_ACT or (fmt == "w8c" and mode is None)
    for M in (32, 33, 48, 49, 64):
        x = synth.activations(6300, M, N, M, K)
        y = _forward(layer, x)
        binding.qfc_tune(9, 64)
        try:
            few = _forward(layer, x)
        finally:
            binding.qfc_tune(9, -1)
        ref = oracle.fc_int8_act(x, wq, s)[3] if int8 else oracle.fc_weight_only(x, wq, s, _group(fmt))
        assert _E(y, ref) <= TOL, M
        if int8:  # exact sums and the same rounding steps
            assert np.array_equal(y.view(np.uint16), few.view(np.uint16)), M
        else:
            assert _E(few, ref) <= TOL, M
    layer.close()


def _launches(call):
    """Kernels that `call` enqueues: the nodes of its captured graph."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    call()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    hip, n = ctypes.CDLL("libamdhip64.so"), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("fmt,pairs,M,N,K,rest", [("w4g32", False, 2698, 3072, 1536, 10), ("w4c", True, 1030, 8192, 2048, 6), ("w4g32", True, 2062, 4096, 1536, 46),
                                                  ("w4c", False, 2698, 3069, 2048, 10), ("w8c", False, 4100, 2045, 1536, 4), ("w4g32", False, 2857, 3072, 2048, 169)])
def test_last_round_of_tiles_left_to_the_token_row_kernels(fmt, pairs, M, N, K, rest):
    """28 x 12 tiles of 96 token rows x 256 channels and the like are a round of 256 workgroups and some more, or end with a tile of few
    rows: the `rest` last rows are computed by the kernels for few token rows, with the residual or the gated output of their rows (rows
    of 2-byte alignment too, more rows than one block of those kernels)."""
    print(f"tail rows {fmt} pairs={pairs} M={M} N={N} K={K}", flush=True)
    wq, s = synth.weights(6200, M, N, synth.FC("t", K, N, fmt))
    x = (synth.activations(6200, M, N, M, K) * np.float16(0.25)).astype(np.float16)
    layer = binding.QuantLinear(wq, s, fmt, compute_mode=binding.QFC_COMPUTE_FP16_DEQUANT, max_m=M, gated_pairs=pairs)
    rows = np.unique(np.concatenate([np.arange(0, M, 97), np.arange(max(0, M - rest - 40), M)]))  # some of all, and both sides of the line
    full = oracle.fc_weight_only(x[rows], wq, s, _group(fmt))
    xd = torch.from_numpy(x).to(DEV)
    guard = torch.full((M + 1, N // 2 if pairs else N), 77.0, dtype=torch.float16, device=DEV)
    if pairs:
        call = lambda: binding.qfc_forward_fused(layer.handle, xd, guard[:M], activation=binding.QFC_ACT_SILU, gated_output=True)
        ref = oracle.gated_output(full, oracle.SILU)
    else:
        res = synth.activations(6201, M, N, M, N)
        rd = torch.from_numpy(res).to(DEV)
        call = lambda: binding.qfc_forward_fused(layer.handle, xd, guard[:M], residual=rd)
        ref = full + res[rows].astype(np.float64)
    assert _launches(call) == 2  # the tiles, then the rows left over
    binding.qfc_tune(9, 0)
    try:
        assert _launches(call) == 1
        one = guard[:M].clone()
    finally:
        binding.qfc_tune(9, -1)
    guard[:M] = 77.0
    call()
    torch.cuda.synchronize()
    # (gated, group scales: the product of two outputs that each carry the rounding of scaled weights, twice the tolerance)
    tol = (2 if pairs and fmt == "w4g32" else 1) * TOL
    assert _E(guard[:M].cpu().numpy()[rows], ref) <= tol
    assert bool((guard[M] == 77.0).all())
    # every row of the two launches against the one launch: each is within the tolerance of the exact result
    a, b = guard[:M].float(), one.float()
    rho = b.pow(2).mean(dim=1, keepdim=True).sqrt()
    assert ((a - b).abs() / torch.maximum(b.abs(), rho)).max().item() <= 2 * tol
    layer.close()


@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,pos0", [(1, 128, 3, 1, 64, 192, 64), (1, 1100, 6, 2, 64, 1152, 13),
                                                   (3, 50, 8, 2, 128, 128, 61), (2, 700, 4, 4, 128, 768, 7), (1, 257, 8, 4, 256, 320, 63),
                                                   # 2, 3, 4, 8 and 2 tokens per workgroup, sequences that end inside one
                                                   (2, 701, 4, 2, 128, 768, 7), (3, 515, 2, 1, 128, 576, 60), (3, 683, 3, 1, 128, 704, 21),
                                                   (3, 1367, 2, 2, 64, 1408, 30), (3, 343, 4, 2, 256, 384, 1),
                                                   # several whole sequences in a workgroup
                                                   (700, 3, 2, 1, 64, 64, 5), (1030, 1, 2, 1, 128, 64, 63),
                                                   # one token per workgroup; both sides of the line by tokens, heads and values
                                                   (3, 50, 16, 8, 128, 128, 61), (1, 128, 24, 8, 128, 192, 64), (1, 319, 8, 1, 128, 384, 9),
                                                   (1, 321, 6, 2, 128, 384, 9)])
def test_rope_qkv_many_tokens(B, S, h_q, h_kv, d, C, pos0):
    """Calls of many values share the evaluation of an angle among the heads of a token: one and
    several tokens per workgroup (at most 512 / d), workgroups that span sequences, cache blocks that the
    tokens fill in part; and the other kernel beside that line."""
    test_rope_qkv_layout(B, S, h_q, h_kv, d, C, pos0)


# the lines at 128 tokens and 400 Ki values, several tokens per workgroup for want of heads, one of 1023 and two of 2048
@pytest.mark.parametrize("B,S,h_q,h_kv,d,C,pos0", [(1, 127, 8, 4, 256, 192, 30), (1, 128, 8, 4, 256, 192, 30), (4, 25, 32, 8, 128, 64, 3),
                                                   (4, 32, 32, 8, 128, 64, 3), (1, 2134, 1, 1, 64, 2176, 1), (1, 1023, 4, 2, 64, 1088, 50),
                                                   (1, 2048, 2, 1, 64, 2112, 50)])
def test_rope_qkv_line_between_kernels(B, S, h_q, h_kv, d, C, pos0):
    test_rope_qkv_layout(B, S, h_q, h_kv, d, C, pos0)


def test_rope_qkv_infinite_values():
    """An infinite or NaN value leaves the rotation as it leaves the definition's: the correction terms of the fp32 pairs
    must not turn an infinity into NaN, not even at position 0, where the sine and its rest are zero."""
    B, S, h_q, h_kv, d, C = 1, 128, 16, 4, 128, 128
    g, W = h_q // h_kv, (h_q + 2 * h_kv) * d
    qkv = synth.activations(3801, 0, 0, S, W).reshape(B, S, W)
    rng = np.random.default_rng(5)
    at = rng.integers(0, qkv.size, 400)
    qkv.reshape(-1)[at] = rng.choice(np.array([np.inf, -np.inf, np.nan, 65504.0, -65504.0], dtype=np.float16), 400)
    q_out = torch.zeros((B * h_kv, S * g, d), dtype=torch.float16, device=DEV)
    kc = torch.zeros((B * h_kv, C, d), dtype=torch.float16, device=DEV)
    vc = torch.zeros((B * h_kv, C // 64, d, 64), dtype=torch.float16, device=DEV)
    binding.qfc_rope_qkv(torch.from_numpy(qkv).to(DEV), 0, _attn_shape(B, h_q, h_kv, d, C), 500000.0, q_out, kc, vc)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        q_ref, k_ref, _ = oracle.rope_qkv_layout(qkv, 0, h_q, h_kv, d, 500000.0)
    for got, ref in ((q_out, q_ref), (kc, k_ref)):
        got = got.cpu().numpy().astype(np.float64).reshape(-1)
        ref = ref.astype(np.float64).reshape(-1)
        odd = ~np.isfinite(ref)
        assert odd.any() and np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(got[odd & ~np.isnan(ref)], ref[odd & ~np.isnan(ref)])


@pytest.mark.parametrize("S,h_q,h_kv,d,base", [(180, 16, 4, 128, 500000.0), (1100, 4, 2, 64, 10000.0), (140, 8, 4, 256, 1e6)])
def test_rope_qkv_both_kernels_give_the_same_bits(S, h_q, h_kv, d, base):
    """The kernel for many tokens, which rotates in pairs of fp32, against the one for few, which does in fp64, on the same tokens in
    calls of 60: every bit, from position 0 on, zeros of both signs, subnormal, largest and infinite values among them
    (and NaN where the other has one)."""
    print(f"rope bits S={S} h_q={h_q} h_kv={h_kv} d={d}", flush=True)
    g, W, C = h_q // h_kv, (h_q + 2 * h_kv) * d, (S + 63) // 64 * 64
    qkv = synth.activations(3802, S, d, S, W)
    rng = np.random.default_rng(d)
    odd = np.array([0.0, -0.0, 6e-8, -6e-8, 3e-5, -6.1e-5, 65504.0, -65504.0, 1.0, -1.0, np.inf, -np.inf, np.nan], dtype=np.float16)
    share = rng.random(qkv.shape)
    qkv = np.where(share < 0.1, rng.choice(odd, qkv.shape), np.where(share < 0.4, rng.choice(odd[:10], qkv.shape), qkv)).astype(np.float16)
    x = torch.from_numpy(qkv).to(DEV)
    shape = _attn_shape(1, h_q, h_kv, d, C)
    outs = []
    for step in (S, 60):
        assert (step < 128) == (step == 60) and (step == 60 or step * W >= 400 << 10)
        kc = torch.zeros((h_kv, C, d), dtype=torch.float16, device=DEV)
        vc = torch.zeros((h_kv, C // 64, d, 64), dtype=torch.float16, device=DEV)
        q = []
        for s0 in range(0, S, step):
            n = min(step, S - s0)
            q.append(torch.zeros((h_kv, n * g, d), dtype=torch.float16, device=DEV))
            binding.qfc_rope_qkv(x[s0:s0 + n].view(1, n, W), s0, shape, base, q[-1], kc, vc)
        torch.cuda.synchronize()
        outs.append([t.cpu().numpy() for t in (torch.cat(q, 1), kc, vc)])
    for many, few in zip(*outs):
        nan = np.isnan(few)
        assert np.array_equal(np.isnan(many), nan) and (few[~nan].view(np.uint16) == 0x8000).any()
        assert np.array_equal(many[~nan].view(np.uint16), few[~nan].view(np.uint16))


def test_native_marshalling_takes_what_the_binding_takes(monkeypatch):
    """The calls that csrc/marshal.cpp lets through give the bits of the other way, and what is not in order is refused alike by both:
    other types, devices, shapes, strides, no rows; subclasses and parameters are taken by both."""
    class Sub(torch.Tensor):
        pass

    N, K, M = 64, 96, 3
    wq, sw = synth.weights(5200, 0, 0, synth.FC("t", K, N, "w8c"))
    layer = _layer(wq, sw, "w8c")
    x = torch.from_numpy(synth.activations(5200, 0, 0, M, K)).to(DEV)
    res = torch.from_numpy(synth.activations(5201, 0, 0, M, N)).to(DEV)
    gamma = torch.ones(K, dtype=torch.float16, device=DEV)
    binding.lib()
    outs = []
    for fast in (binding._fast, None):
        monkeypatch.setattr(binding, "_fast", fast)
        for xx in (x, x.as_subclass(Sub), torch.nn.Parameter(x, requires_grad=False)):
            y, z = (torch.empty((M, N), dtype=torch.float16, device=DEV) for _ in range(2))
            binding.qfc_forward(layer.handle, xx, y)
            binding.qfc_forward_fused(layer.handle, xx, z, residual=res, norm_gamma=gamma, norm_eps=1e-5, norm_offset=1)
            outs.append(torch.stack([y, z]))
        y = torch.empty((M, N), dtype=torch.float16, device=DEV)
        wide = torch.zeros((M, 2 * K), dtype=torch.float16, device=DEV)
        for bad in (x.float(), x.cpu(), x[:, :32], wide[:, ::2], x[0], None, x.view(M, K, 1)):
            with pytest.raises(ValueError):
                binding.qfc_forward(layer.handle, bad, y)
            with pytest.raises(ValueError):
                binding.qfc_forward_fused(layer.handle, bad, y, residual=res)
        for kw in (dict(residual=res[:2]), dict(residual=res.float()), dict(norm_gamma=gamma[:32]), dict(gate=res)):
            with pytest.raises(ValueError):
                binding.qfc_forward_fused(layer.handle, x, y, **kw)
        with pytest.raises(ValueError):
            binding.qfc_forward(layer.handle, x, y[:2])
        with pytest.raises(binding.QfcError):
            binding.qfc_forward(layer.handle, x[:0], y[:0])
        with pytest.raises(binding.QfcError):  # 2 bytes off the 16 that the library asks for
            off = torch.zeros(M * K + 1, dtype=torch.float16, device=DEV)[1:].view(M, K)
            binding.qfc_forward(layer.handle, off, y)
    torch.cuda.synchronize()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])
    layer.close()


def test_native_marshalling_takes_the_calls_in_order():
    """What csrc/marshal.cpp itself says: plain tensors and parameters in order go through it (status 0), subclasses and anything that is not in
    order do not (-1); with a gate and with a gated output it gives the bits of the other way."""
    class Sub(torch.Tensor):
        pass

    N, K, M = 64, 96, 3
    wq, sw = synth.weights(5210, 0, 0, synth.FC("t", K, N, "w8c"))
    layer = _layer(wq, sw, "w8c")
    pairs = binding.QuantLinear(wq, sw, "w8c", max_m=M, gated_pairs=True)
    x, gate = (torch.from_numpy(synth.activations(5210 + i, 0, 0, M, K)).to(DEV) for i in range(2))
    res = torch.from_numpy(synth.activations(5212, 0, 0, M, N)).to(DEV)
    gamma = torch.ones(K, dtype=torch.float16, device=DEV)
    y = torch.empty((M, N), dtype=torch.float16, device=DEV)
    fast = binding._fast
    assert fast is not None

    def plain(xx, yy):
        return fast.forward(layer.handle.value, xx, yy, N, K)

    def fused(xx, yy, l=layer, gate=None, act=0, residual=None, gated=False, gamma=None):
        return fast.forward_fused(l.handle.value, xx, yy, N, K, gate, act, residual, gated, gamma, 1e-5, 0)

    half = torch.empty((M, N // 2), dtype=torch.float16, device=DEV)
    assert plain(x, y) == 0 and plain(torch.nn.Parameter(x, requires_grad=False), y) == 0 and fused(x, y) == 0
    assert fused(x, y, gate=gate, act=binding.QFC_ACT_GELU_TANH) == 0 and fused(x, y, residual=res, gamma=gamma) == 0
    assert fused(x, half, l=pairs, gated=True) == 0
    assert plain(x[:0], y[:0]) == -1 and fused(x[:0], y[:0]) == -1
    off = torch.zeros(M * K + 1, dtype=torch.float16, device=DEV)[1:].view(M, K)
    assert plain(off, y) == binding.QFC_ERR_ALIGNMENT and fused(off, y) == binding.QFC_ERR_ALIGNMENT
    wide = torch.zeros((M, 2 * K), dtype=torch.float16, device=DEV)
    for bad in (x.as_subclass(Sub), x.float(), x.cpu(), x[:, :32], wide[:, ::2], x[0], None, x.view(M, K, 1), x[:2]):
        assert plain(bad, y) == -1 and fused(bad, y) == -1
        if bad is not None:
            assert fused(x, y, gate=bad) == -1
    for bad in (y[:2], y.float(), half, None):
        assert plain(x, bad) == -1 and fused(x, bad) == -1
        if bad is not None:
            assert fused(x, y, residual=bad) == -1
    for bad in (gamma[:32], gamma.float(), gamma.view(1, K), gamma.as_subclass(Sub)):
        assert fused(x, y, gamma=bad) == -1
    assert fused(x, y, l=pairs, gated=True) == -1 and fused(x, half, l=pairs, gated=True, residual=res) == -1
    assert fused(x, y, act=0.5) == -1 and fused(x, y, act=1 << 31) == -1

    def both(f):
        outs = []
        for way in (fast, None):
            binding._fast = way
            outs.append(f().clone())
        return torch.equal(*outs)

    try:
        assert both(lambda: (binding.qfc_forward_fused(layer.handle, x, y, gate=gate, activation=binding.QFC_ACT_GELU_TANH), y)[1])
        assert both(lambda: (binding.qfc_forward_fused(layer.handle, x, y, gate=gate, residual=res), y)[1])
        assert both(lambda: (binding.qfc_forward_fused(pairs.handle, x, half, gated_output=True, norm_gamma=gamma, norm_eps=1e-5), half)[1])
    finally:
        binding._fast = fast
    layer.close()
    pairs.close()


# more KV heads than compute units, one walk each and four, 16 and 8 query rows per head, all head sizes (head size 256: walks of 32 positions)
@pytest.mark.parametrize("G,M,d,n_ctx", [(257, 16, 256, 1084), (257, 16, 256, 1083), (258, 8, 128, 900), (257, 16, 64, 1100), (262, 5, 256, 1000), (520, 3, 64, 1301)])
def test_attention_many_heads_and_rows_sampled(G, M, d, n_ctx):
    """Sampled KV heads, the first and the last among them, against the oracle; the call's own number of walks and one."""
    print(f"attention G={G} M={M} d={d} n_ctx={n_ctx}", flush=True)
    C = (n_ctx + 63) // 64 * 64
    gen = torch.Generator(device=DEV)
    gen.manual_seed(G + n_ctx)
    q, kc, vc = (torch.randn(s, generator=gen, device=DEV).half() for s in ((G, M, d), (G, C, d), (G, C // 64, d, 64)))
    shape = _attn_shape(G, M, 1, d, C)
    ws = torch.empty(binding.qfc_attention_workspace_size(shape, 1), dtype=torch.uint8, device=DEV)
    heads = sorted({0, G - 1, *np.random.default_rng(G).integers(0, G, 6).tolist()})
    ref = oracle.attention(q[heads].cpu().numpy(), kc[heads].cpu().numpy(), binding.vcache_logical(vc[heads]).cpu().numpy(), n_ctx, 1)
    for walks in (0, 1):
        out = torch.full((G, M, d), 7.0, dtype=torch.float16, device=DEV)
        binding.qfc_tune(12, walks)
        try:
            binding.qfc_attention(q, kc, vc, 1, n_ctx, shape, ws, out)
            torch.cuda.synchronize()
        finally:
            binding.qfc_tune(12, 0)
        assert not (out == 7.0).all(-1).any()
        assert _E(out[heads].cpu().numpy().reshape(-1, d), ref.reshape(-1, d)) <= TOL, walks
