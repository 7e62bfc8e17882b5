"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Gates: sign pack/unpack bit-exact; y within max|Y-Y*|/max|Y*| <= 2e-3 (fp16 staging, fp32
accumulation); the fp32 ("precise") path within 2e-5; exact-integer inputs bit-for-bit."""
import numpy as np
import pytest

from oracle import mdbf_oracle as orc
from paper_2512_24545_amd import synth
from helpers import concat_terms

pytestmark = pytest.mark.gpu

TOL = 2e-3
TOL_PRECISE = 2e-5


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2512_24545_amd import binding as mb
    mb.lib()
    return torch, mb


def _oracle_args(L):
    return (L["SA"], L["SB"], L["A"], L["Q"], L["G"], L["B"])


def _to_dev(torch, X, dtype):
    t = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    return torch.from_numpy(np.ascontiguousarray(X)).to("cuda:0").to(t).contiguous()


def _run(gpu, L, X, x_dtype, y_dtype="f32", precise=False, block_scaled=False):
    torch, mb = gpu
    dl = mb.DeviceLayer.from_host(L)
    Xd = _to_dev(torch, X, x_dtype)
    Y = mb.mdbf_forward(dl, Xd, y_dtype=y_dtype, precise=precise, block_scaled=block_scaled)
    torch.cuda.synchronize()
    return Y.float().cpu().numpy().astype(np.float64)


# ---------------------------------------------------------------- pack / unpack
@pytest.mark.parametrize("rows,cols", [(1, 1), (16, 128), (17, 129), (5, 31), (33, 500), (100, 1000),
                                       (256, 128), (2656, 4096), (4096, 2656)])
def test_pack_unpack_bit_exact(gpu, rows, cols):
    torch, mb = gpu
    rng = np.random.default_rng(rows * 7919 + cols)
    S = synth.random_signs(rng, rows, cols)
    Sd = torch.from_numpy(S).to("cuda:0")
    packed = mb.mdbf_pack(Sd)
    assert packed.numel() == mb.mdbf_packed_bytes(rows, cols)
    back = mb.mdbf_unpack(packed, rows, cols).cpu().numpy()
    np.testing.assert_array_equal(back, S)
    # the logical bits agree with the oracle's reference packing of the same matrix
    np.testing.assert_array_equal(orc.unpack_ref(orc.pack_ref(S), cols), back)
    # one bit per entry, padding bits are zero: population count equals the number of -1 entries
    pc = int(np.unpackbits(packed.cpu().numpy()).sum())
    assert pc == int((S < 0).sum())


def test_pack_zero_is_plus_and_strided_input(gpu):
    torch, mb = gpu
    rng = np.random.default_rng(5)
    big = rng.integers(-3, 4, size=(40, 300)).astype(np.int8)   # includes zeros and |v| > 1
    view = torch.from_numpy(big).to("cuda:0")[:, 10:210]          # leading dimension 300 > cols 200
    packed = mb.mdbf_pack(view)
    back = mb.mdbf_unpack(packed, 40, 200).cpu().numpy()
    np.testing.assert_array_equal(back, orc.sign_pm1(big[:, 10:210]))


@pytest.mark.parametrize("rows,cols,pad", [(16, 512, 0), (63, 513, 3), (65, 1023, 5), (1041, 519, 1), (33, 1536, 7), (3, 7, 2)])
def test_packed_words_are_where_the_layout_says(gpu, rows, cols, pad):
    """Every word of the packed blob, from the layout's formula, at the edges of the packing kernel's blocks of
    512 columns, of its 8-column groups and of a group of 64 tiles, with rows at any byte alignment."""
    torch, mb = gpu
    rng = np.random.default_rng(rows + cols)
    big = torch.from_numpy(rng.integers(-2, 2, size=(rows, cols + 2 * pad)).astype(np.int8)).to("cuda:0")
    view = big[:, pad:pad + cols]
    neg = view.cpu().numpy() < 0
    nt, nb = (rows + 15) // 16, (cols + 127) // 128
    full = np.zeros((nt * 16, nb * 128), dtype=bool)
    full[:rows, :cols] = neg
    want = np.zeros(nt * nb * 64, dtype=np.uint32)
    kl = np.arange(128)
    f, e = kl // 32, kl % 8
    bit = (8 * (f // 2) + 4 * (f % 2) + e // 2 + 16 * (e % 2)).astype(np.uint32)
    for t in range(nt):
        g0 = t // 64 * 64
        gt = min(64, nt - g0)
        for q in range(nb):
            blk = full[t * 16:t * 16 + 16, q * 128:q * 128 + 128].astype(np.uint32) << bit
            for kg in range(4):
                base = (g0 * nb + q * gt + (t - g0)) * 64 + kg * 16
                want[base:base + 16] = np.bitwise_or.reduce(blk[:, (kl % 32) // 8 == kg], axis=1)
    packed = mb.mdbf_pack(view)
    np.testing.assert_array_equal(packed.cpu().numpy().view(np.uint32), want)
    np.testing.assert_array_equal(mb.mdbf_unpack(packed, rows, cols).cpu().numpy() < 0, neg)


@pytest.mark.parametrize("rows,cols,first,pitch", [(1, 512, 1, 515), (16, 1024, 0, 1024), (17, 511, 3, 700), (37, 1537, 5, 1543), (70, 1151, 0, 1151)])
def test_pack_runs_of_blocks_at_any_alignment(gpu, rows, cols, first, pitch):
    """Whole runs of four blocks (through LDS) and cut ones, rows at odd addresses, the last row at the end of the buffer,
    rows that do not fill the last tile; what lies between the rows is neither packed nor written."""
    torch, mb = gpu
    L = mb.lib()
    rng = np.random.default_rng(rows + cols)
    S = synth.random_signs(rng, rows, cols)
    buf = torch.full((first + (rows - 1) * pitch + cols,), -7, dtype=torch.int8, device="cuda:0")
    view = buf[first:].as_strided((rows, cols), (pitch, 1))
    view.copy_(torch.from_numpy(S))
    packed = mb.mdbf_pack(view)
    assert torch.equal(packed, mb.mdbf_pack(torch.from_numpy(S).cuda()))
    back = torch.full_like(buf, -7)
    stream = torch.cuda.current_stream().cuda_stream
    assert L.mdbf_unpack(packed.data_ptr(), rows, cols, back[first:].data_ptr(), pitch, stream) == 0
    assert torch.equal(back, buf)
    np.testing.assert_array_equal(mb.mdbf_unpack(packed, rows, cols).cpu().numpy(), S)


@pytest.mark.parametrize("cols", [2 ** 31 - 128, 2 ** 31 - 131])
def test_pack_a_row_near_the_largest_int(gpu, cols):
    """The last blocks of a row whose padded end is no int any more: what lies behind the row (negative bytes: bits
    that would be set) is neither packed nor written."""
    torch, mb = gpu
    if torch.cuda.get_device_properties(0).total_memory < 32 << 30:
        pytest.skip("needs four buffers of 2 GiB")
    buf = torch.full((cols + 4096,), -1, dtype=torch.int8, device="cuda:0")
    buf[:cols] = 1
    where = torch.cat([torch.arange(0, cols, 9973, device="cuda:0"), torch.tensor([cols - 1, cols - 7, cols - 600], device="cuda:0")])
    buf[where] = -1
    packed = mb.mdbf_pack(buf[:cols].view(1, cols))
    words = packed.view(torch.int32)
    assert words.numel() == (2 ** 24 - 1) * 64
    got = sum(int((words >> b & 1).sum()) for b in range(32))
    assert got == torch.unique(where).numel()
    back = torch.full_like(buf, -1)
    L = mb.lib()
    assert L.mdbf_unpack(packed.data_ptr(), 1, cols, back.data_ptr(), cols, torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(back, buf)


# ---------------------------------------------------------------- forward: small and ragged
SMALL = [
    # m, n, k, l, T
    (16, 128, 16, 16, 1),
    (256, 256, 128, 4, 1),
    (40, 300, 70, 16, 2),
    (130, 129, 257, 3, 3),
    (1, 1, 1, 1, 1),
    (100, 1030, 200, 8, 1),
    (530, 2100, 1100, 16, 2),
    (77, 64, 2656, 2, 1),
]


@pytest.mark.parametrize("nbytes,waves", [(16, 4), (16 * 1000, 4), (16 * 65537, 64), (1 << 22, 8192), ((1 << 22) + 48, 1028)])
def test_stream_read_folds_every_word_once(gpu, nbytes, waves):
    """The bandwidth yardstick reads every 16-byte element exactly once: the XOR of its per-wave words equals
    the XOR of all 32-bit words of the buffer, for sizes below, equal to and far above one trip of the launch."""
    torch, mb = gpu
    rng = np.random.default_rng(nbytes % 1000 + waves)
    host = rng.integers(0, 2 ** 32, size=nbytes // 4, dtype=np.uint32)
    src = torch.from_numpy(host.view(np.int32)).to("cuda:0")
    sink = torch.full((waves,), 0x5A5A5A5A, dtype=torch.int32, device="cuda:0")
    mb.mdbf_stream_read(src, sink)
    torch.cuda.synchronize()
    got = np.bitwise_xor.reduce(sink.cpu().numpy().view(np.uint32))
    assert got == np.bitwise_xor.reduce(host)


@pytest.mark.parametrize("m,n,k,l,T", SMALL)
@pytest.mark.parametrize("precise", [False, True])
def test_forward_small_shapes(gpu, m, n, k, l, T, precise):
    L = synth.make_layer(m, n, k, l, seed=m + 3 * n + 5 * k + l, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=99 + m, x_dtype="f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32", precise)
    err = orc.max_rel_error(got, ref)
    assert err <= (TOL_PRECISE if precise else TOL), err


@pytest.mark.parametrize("env_dtype,x_dtype,y_dtype", [("f32", "f32", "f32"), ("bf16", "bf16", "f32"),
                                                         ("f16", "f16", "f16"), ("f16", "bf16", "bf16"),
                                                         ("f32", "f16", "f32")])
def test_forward_dtypes(gpu, env_dtype, x_dtype, y_dtype):
    L = synth.make_layer(96, 200, 150, 5, seed=17, env_dtype=env_dtype, env_kind="llama", signed_env=True)
    X = synth.make_activations(200, 2, seed=18, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, x_dtype, y_dtype)
    # a 16-bit output adds its own rounding: half an ulp of the largest element
    slack = {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[y_dtype]
    assert orc.max_rel_error(got, ref) <= TOL + slack


def test_toy_config(gpu):
    """256x256, k=128, l=4, fp32 envelopes and activations."""
    L, X = synth.config_toy()
    ref = orc.forward_dense(*_oracle_args(L), X)
    np.testing.assert_allclose(orc.forward_factored(*_oracle_args(L), X), ref, rtol=1e-10, atol=1e-9)
    for precise, tol in ((False, TOL), (True, TOL_PRECISE)):
        got = _run(gpu, L, X, "f32", "f32", precise)
        assert orc.max_rel_error(got, ref) <= tol


# ---------------------------------------------------------------- exact-integer inputs: zero tolerance
@pytest.mark.parametrize("m,n,k,l", [(64, 256, 96, 4), (530, 2100, 1100, 16), (4096, 4096, 2656, 4)])
def test_exact_integer_inputs_bit_for_bit(gpu, m, n, k, l):
    """All-ones envelopes and x in {-1,0,1}: every intermediate is an integer that fp16 staging and
    fp32 accumulation represent exactly, so the result must equal the oracle in any summation order."""
    L = synth.make_layer(m, n, k, l, seed=31 + m, env_dtype="f16", env_kind="ones")
    X = synth.make_activations(n, 1, seed=32, x_dtype="f16", kind="ternary")
    ref = orc.forward_factored(*_oracle_args(L), X)
    assert np.max(np.abs(ref)) < 2 ** 24
    got = _run(gpu, L, X, "f16", "f32")
    np.testing.assert_array_equal(got, ref)


# ---------------------------------------------------------------- the block-scaled variant, forced
# (without the flag the library takes it only for launches that fill the device: the bench-sized plans)
BLOCK_SCALED = [
    # m, n, k, T: ragged K, one or many stages, partial tile groups, several items per matrix
    (16, 128, 16, 1),
    (40, 300, 70, 2),
    (530, 2100, 1100, 3),
    (1100, 1030, 2105, 1),
    (2064, 520, 4100, 16),
    (4096, 4096, 2656, 1),
]


@pytest.mark.parametrize("m,n,k,T", BLOCK_SCALED)
def test_block_scaled_shapes(gpu, m, n, k, T):
    L = synth.make_layer(m, n, k, 16, seed=m + 3 * n + 5 * k, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=77 + m, x_dtype="f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32", block_scaled=True)
    assert orc.max_rel_error(got, ref) <= TOL


@pytest.mark.parametrize("m,n,k,T", [(40, 300, 70, 2), (1100, 1030, 2105, 1), (4096, 4096, 1856, 1), (2064, 520, 4100, 16)])
def test_block_scaled_rank_8(gpu, m, n, k, T):
    """Rank-8 envelopes (the 1.0 bits-per-weight budget) through the block-scaled kernel: the 16-wide
    matrix-core tile carries two limbs of every mode side by side."""
    L = synth.make_layer(m, n, k, 8, seed=m + 3 * n + 5 * k + 8, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=78 + m, x_dtype="f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32", block_scaled=True)
    assert orc.max_rel_error(got, ref) <= TOL


@pytest.mark.parametrize("x_dtype,y_dtype", [("bf16", "bf16"), ("f32", "f32"), ("f16", "f16")])
def test_block_scaled_dtypes(gpu, x_dtype, y_dtype):
    L = synth.make_layer(300, 700, 450, 16, seed=23, env_dtype="f16", env_kind="llama", signed_env=True)
    X = synth.make_activations(700, 2, seed=24, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, x_dtype, y_dtype, block_scaled=True)
    slack = {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[y_dtype]
    assert orc.max_rel_error(got, ref) <= TOL + slack


@pytest.mark.parametrize("m,n,k", [(64, 256, 96), (530, 2100, 1100), (4096, 4096, 2656)])
def test_block_scaled_exact_integer_inputs(gpu, m, n, k):
    """All-ones envelopes (l = 16) and x in {-1,0,1}: the scaled activations are small integers times a
    power of two, which three fp6 limbs under a shared exponent hold exactly; fp32 accumulation is exact
    below 2^24.  The result must equal the oracle bit for bit."""
    L = synth.make_layer(m, n, k, 16, seed=41 + m, env_dtype="f16", env_kind="ones")
    X = synth.make_activations(n, 1, seed=42, x_dtype="f16", kind="ternary")
    ref = orc.forward_factored(*_oracle_args(L), X)
    assert np.max(np.abs(ref)) < 2 ** 24
    got = _run(gpu, L, X, "f16", "f32", block_scaled=True)
    np.testing.assert_array_equal(got, ref)


def test_block_scaled_batch_equals_single_calls(gpu):
    torch, mb = gpu
    specs = [(530, 2104, 1104, 2), (4096, 4096, 2656, 1), (272, 1032, 4096, 16), (1100, 1030, 2105, 1)]
    layers, Xs, Ys, refs, singles = [], [], [], [], []
    for i, (m, n, k, T) in enumerate(specs):
        L = synth.make_layer(m, n, k, 16, seed=300 + i, env_dtype="f16", env_kind="llama", signed_env=True)
        X = synth.make_activations(n, T, seed=400 + i, x_dtype="f16")
        dl = mb.DeviceLayer.from_host(L)
        Xd = _to_dev(torch, X, "f16")
        layers.append(dl)
        Xs.append(Xd)
        Ys.append(torch.zeros((T, m), dtype=torch.float32, device="cuda:0"))
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        singles.append(mb.mdbf_forward(dl, Xd, y_dtype="f32", block_scaled=True))
    plan = mb.BatchPlan(layers, Xs, Ys, block_scaled=True)
    plan.run()
    torch.cuda.synchronize()
    for (m, n, k, T), Yb, Y1, ref in zip(specs, Ys, singles, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL
        if T == 1:
            # a single call with one token splits the contraction across workgroups: fp32 partial sums added
            # in another (fixed) order, so z differs in its last bits and a few of its limbs round the other way
            assert orc.max_rel_error(Yb.cpu().numpy(), Y1.cpu().numpy().astype(np.float64)) <= 5e-4
        else:
            assert torch.equal(Yb, Y1)


# ---------------------------------------------------------------- LLaMA-7B shaped layers
def test_attention_projection_decode(gpu):
    """4096x4096, k=2656, l=16, one fp16 token (about 1.5 bits per weight)."""
    L, X = synth.config_attn_decode()
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32")
    assert orc.max_rel_error(got, ref) <= TOL
    got16 = _run(gpu, L, X, "f16", "f16")
    assert orc.max_rel_error(got16, ref) <= TOL + 2.0 ** -11


@pytest.mark.parametrize("which", ["gate", "down"])
@pytest.mark.parametrize("T", [1, 16])
def test_mlp_projections_decode(gpu, which, T):
    L, X = synth.config_mlp_decode(which, T=T)
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32")
    assert orc.max_rel_error(got, ref) <= TOL


def test_determinism(gpu):
    torch, mb = gpu
    L, X = synth.config_attn_decode(seed=7, T=2)
    dl = mb.DeviceLayer.from_host(L)
    Xd = _to_dev(torch, X, "f16")
    Y1 = mb.mdbf_forward(dl, Xd).clone()
    Y2 = mb.mdbf_forward(dl, Xd)
    torch.cuda.synchronize()
    assert torch.equal(Y1, Y2)


def test_determinism_of_the_split_contraction(gpu):
    """One token: the contraction of each factor is split across workgroups and the partial sums are added in a
    fixed order (by the reader for the first factor, by the last workgroup to finish for the second), so
    repeated calls give the same bits, whichever workgroup finishes last."""
    torch, mb = gpu
    for seed, (m, n, k, l) in enumerate([(4096, 4096, 2656, 16), (1100, 1030, 2105, 16), (530, 2104, 1104, 8)]):
        L = synth.make_layer(m, n, k, l, seed=70 + seed, env_dtype="f16", env_kind="llama", signed_env=True)
        X = synth.make_activations(n, 1, seed=80 + seed, x_dtype="f16")
        dl = mb.DeviceLayer.from_host(L)
        Xd = _to_dev(torch, X, "f16")
        first = mb.mdbf_forward(dl, Xd, y_dtype="f32").clone()
        for _ in range(20):
            again = mb.mdbf_forward(dl, Xd, y_dtype="f32")
            assert torch.equal(first, again)
        ref = orc.forward_factored(*_oracle_args(L), X)
        assert orc.max_rel_error(first.cpu().numpy(), ref) <= TOL


FEW_TOKENS = [
    # m, n, k, l, T, env, x, columns of X behind each row: rows shorter than a vector, last octets of 1 and 7 columns,
    # chunk and split edges, the largest token count of each slab count, rows at odd addresses
    (5, 3, 7, 1, 2, "f32", "f32", 0), (16, 129, 127, 16, 16, "f16", "bf16", 3), (130, 513, 1031, 8, 7, "f16", "f32", 1),
    (1041, 4097, 2049, 3, 17, "bf16", "f16", 5), (300, 1025, 4100, 15, 32, "f32", "bf16", 0),
    (2064, 2055, 515, 5, 33, "f16", "f32", 2), (4096, 11008, 4096, 16, 16, "f16", "f16", 8), (520, 640, 3000, 16, 64, "f32", "f16", 1),
]


@pytest.mark.parametrize("m,n,k,l,T,env_dtype,x_dtype,pad", FEW_TOKENS)
def test_few_token_calls(gpu, m, n, k, l, T, env_dtype, x_dtype, pad):
    """Single calls with 2 to 64 tokens, the contraction split across workgroups and (with a workspace that has no
    room for partial sums) in one run: both against the oracle at the fp16 gate, and against each other: z is
    rounded to fp16 between the factors, so a sum that rounds the other way moves it by 2^-11."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l + T, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=19 + m, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    dl = mb.DeviceLayer.from_host(L)
    wide = torch.full((T, n + pad), float("nan"), dtype=_to_dev(torch, X[:1], x_dtype).dtype, device="cuda:0")
    wide[:, :n] = _to_dev(torch, X, x_dtype)
    Xd = wide[:, :n]
    got = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    assert orc.max_rel_error(got.cpu().numpy(), ref) <= TOL
    assert torch.equal(got, mb.mdbf_forward(dl, Xd, y_dtype="f32"))
    assert torch.equal(mb.mdbf_forward(dl, Xd, y_dtype="f32", Y=got.clone(), accumulate=True), got + got)
    z = (T * ((k + 7) // 8 * 8) * 4 + 255) // 256 * 256
    small = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32", precise=True), T), dtype=torch.uint8, device="cuda:0")
    assert small.numel() == z
    if T > 16 or l not in (8, 16) or env_dtype != "f16":
        run = mb.mdbf_forward(dl, Xd, y_dtype="f32", workspace=small)
        assert orc.max_rel_error(run.cpu().numpy(), ref) <= TOL
        assert orc.max_rel_error(run.cpu().numpy(), got.cpu().numpy().astype(np.float64)) <= 2.0 ** -11


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", [
    (5000, 3001, 2003, 3, "bf16", "bf16"), (9920, 640, 1790, 3, "f16", "f16"), (9920, 896, 1792, 16, "f16", "f16")])
def test_a_token_of_a_short_call_does_not_depend_on_its_length(gpu, m, n, k, l, env_dtype, x_dtype):
    """The split of the contraction is one for 2 to 16 tokens and one for 17 to 64: the same bits in every call of a
    range.  Shapes whose best split, priced by the token count, would change inside of one."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    dl = mb.DeviceLayer.from_host(L)
    X = _to_dev(torch, synth.make_activations(n, 64, seed=5, x_dtype=x_dtype), x_dtype)
    for lo, hi in ((2, 16), (17, 64)):
        full = mb.mdbf_forward(dl, X[:hi], y_dtype="f32")
        for T in sorted({lo, lo + 1, (lo + hi) // 2, 32, 33, hi - 1} & set(range(lo, hi))):
            assert torch.equal(mb.mdbf_forward(dl, X[:T], y_dtype="f32"), full[:T]), T


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", [(300, 649, 1515, 12, "f32", "f32"), (530, 1027, 300, 3, "bf16", "bf16"), (65, 7, 130, 16, "f16", "f16")])
def test_short_calls_of_any_number_of_slabs(gpu, m, n, k, l, env_dtype, x_dtype):
    """17 to 64 tokens in two, three and four slabs of sixteen, the last one full and with a single token: the bits of 64
    tokens, which meet the oracle at the fp16 gate; rows apart by one element more than they have."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    dl, X = mb.DeviceLayer.from_host(L), synth.make_activations(n, 64, seed=5, x_dtype=x_dtype)
    wide = torch.full((64, n + 1), float("nan"), dtype=_to_dev(torch, X[:1], x_dtype).dtype, device="cuda:0")
    wide[:, :n] = _to_dev(torch, X, x_dtype)
    full = mb.mdbf_forward(dl, wide[:, :n], y_dtype="f32")
    assert orc.max_rel_error(full.cpu().numpy(), orc.forward_factored(*_oracle_args(L), X)) <= TOL
    for T in (17, 32, 33, 48, 49):
        assert torch.equal(mb.mdbf_forward(dl, wide[:T, :n], y_dtype="f32"), full[:T]), T


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", [
    (5000, 3001, 2003, 3, "bf16", "bf16"), (2064, 1032, 2056, 16, "f16", "f16"), (300, 649, 1515, 12, "f32", "f32")])
def test_a_longer_calls_workspace_serves_the_shorter_ones_alike(gpu, m, n, k, l, env_dtype, x_dtype):
    """One buffer, sized for 130 tokens: every shorter call returns the bits it returns with a buffer of its own."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    dl = mb.DeviceLayer.from_host(L)
    X = _to_dev(torch, synth.make_activations(n, 130, seed=5, x_dtype=x_dtype), x_dtype)
    ws = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32"), 130), dtype=torch.uint8, device="cuda:0")
    for T in (1, 2, 16, 17, 40, 64, 65, 128):
        got = mb.mdbf_forward(dl, X[:T], y_dtype="f32", workspace=ws)
        assert torch.equal(got, mb.mdbf_forward(dl, X[:T], y_dtype="f32")), T


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype,pad", [
    (530, 1032, 1000, 16, "f16", "f16", 8), (2064, 520, 1160, 8, "f16", "bf16", 1), (300, 649, 515, 3, "bf16", "bf16", 0),
    (130, 1025, 2049, 16, "f32", "f32", 3), (17, 5, 9, 1, "f32", "f16", 1)])
def test_a_token_of_a_long_call_does_not_depend_on_its_length(gpu, m, n, k, l, env_dtype, x_dtype, pad):
    """From 65 tokens on every token is the same sum in the same order, whatever tile shape the call's length
    picks and whether the operands are loaded as they are or copied to fp16 first (without room for the copies:
    element by element): the same bits.  The longest call against the oracle at the fp16 gate."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 2100, seed=29 + m, x_dtype=x_dtype)
    dl = mb.DeviceLayer.from_host(L)
    wide = torch.full((2100, n + pad), float("nan"), dtype=_to_dev(torch, X[:1], x_dtype).dtype, device="cuda:0")
    wide[:, :n] = _to_dev(torch, X, x_dtype)
    Xd = wide[:, :n]
    full = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    rows = list(range(0, 2100, 171))
    assert orc.max_rel_error(full[rows].cpu().numpy(), orc.forward_factored(*_oracle_args(L), X[rows])) <= TOL
    for T in (65, 97, 128, 300, 777, 1500):
        assert torch.equal(mb.mdbf_forward(dl, Xd[:T], y_dtype="f32"), full[:T]), T
    ws = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32", precise=True), 777), dtype=torch.uint8, device="cuda:0")
    assert torch.equal(mb.mdbf_forward(dl, Xd[:777], y_dtype="f32", workspace=ws), full[:777])
    assert torch.equal(mb.mdbf_forward(dl, Xd[:777], y_dtype="f32", Y=full[:777].clone(), accumulate=True), full[:777] * 2)


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", [
    (90, 300, 203, 3, "bf16", "bf16"), (90, 256, 40, 16, "f16", "f32"), (17, 5, 9, 1, "f32", "f16"), (40, 130, 128, 8, "f32", "f32")])
def test_overflows_of_a_long_call_do_not_depend_on_the_copies(gpu, m, n, k, l, env_dtype, x_dtype):
    """One entry of the first token's z overflows fp16 (its row of G is 2^12 times the others): its outputs are
    infinities with the fp16 copies as without room for them, element by element, and the other tokens are the same
    bits.  Entries in the last, partial block and octet of z above all."""
    torch, mb = gpu
    T = 70
    L = synth.make_layer(m, n, k, l, seed=m + k, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=4, x_dtype=x_dtype)
    for j in sorted({0, k // 2, k - 1, k - 2, max(0, k - 9)}):
        H = dict(L, G=L["G"] * 2.0 ** -6)
        H["G"][j] = L["G"][j] * 2.0 ** 6
        z = H["G"][j] @ ((L["SB"][j][:, None] * L["B"]).T @ X[0])
        Xj = X.copy()
        Xj[0] *= 2.0 ** np.ceil(np.log2(4 * 65504 / abs(z)))
        dl, Xd = mb.DeviceLayer.from_host(H), _to_dev(torch, Xj, x_dtype)
        small = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32", precise=True), T), dtype=torch.uint8, device="cuda:0")
        got = mb.mdbf_forward(dl, Xd, y_dtype="f32").cpu().numpy()
        want = mb.mdbf_forward(dl, Xd, y_dtype="f32", workspace=small).cpu().numpy()
        assert np.isinf(want[0]).all() and np.isfinite(want[1:]).all(), j
        np.testing.assert_array_equal(got, want)


ANY_RANK = [
    # m, n, k, l, env, x: edges of the 16-row tiles, of the 128-column blocks, of the 8-tile groups and of a split of
    # four blocks; the smallest and largest rank of both record forms
    (1, 1, 1, 1, "f32", "f32"), (16, 127, 128, 8, "bf16", "f16"), (17, 129, 127, 9, "f16", "bf16"),
    (129, 513, 385, 1, "f16", "f16"), (128, 512, 1024, 16, "f32", "f32"), (2049, 4097, 1601, 3, "bf16", "bf16"),
    (300, 5000, 2049, 15, "f32", "f16"),
]


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", ANY_RANK)
def test_one_token_calls_of_any_rank_and_type(gpu, m, n, k, l, env_dtype, x_dtype):
    """fp32 throughout (the gate of 1e-4 is wider than that needs: test_one_token_calls_are_fp32 has the narrow one).  A
    workspace without room for partial sums takes the fp16-staged general kernel instead; an infinity or NaN
    anywhere in the input reaches every output."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="llama", signed_env=True)
    X = synth.make_activations(n, 1, seed=9 + m, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, x_dtype)
    got = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    assert orc.max_rel_error(got.cpu().numpy(), ref) <= 1e-4
    assert torch.equal(got, mb.mdbf_forward(dl, Xd, y_dtype="f32"))
    twice = mb.mdbf_forward(dl, Xd, y_dtype="f32", Y=got.clone(), accumulate=True)
    assert torch.equal(twice, got + got)
    small = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32", fp16_staged=True), 1), dtype=torch.uint8, device="cuda:0")
    if l not in (8, 16) or env_dtype != "f16":
        staged = mb.mdbf_forward(dl, Xd, y_dtype="f32", workspace=small)
        assert torch.equal(staged, mb.mdbf_forward(dl, Xd, y_dtype="f32", fp16_staged=True))
    for where in {0, n // 2, n - 1}:
        for bad in (float("inf"), float("nan")):
            Xb = Xd.clone()
            Xb[0, where] = bad
            assert not torch.isfinite(mb.mdbf_forward(dl, Xb, y_dtype="f32")).any()


ONE_TOKEN_EDGES = [
    # m, n, k, l, env, x: factors of fewer elements than a vector; last vectors that begin before the last block; rows that
    # end in the middle of one, for each number of modes a lane holds; blocks on one to four workgroups and on 1 to 16
    # waves, one to six blocks a wave
    (3, 2, 1, 3, "f16", "f16"), (17, 1, 5, 1, "bf16", "bf16"), (16, 129, 257, 1, "f16", "bf16"), (40, 130, 3, 7, "bf16", "f16"),
    (33, 257, 1030, 9, "f16", "f32"), (31, 385, 129, 15, "bf16", "f32"), (90, 130, 129, 2, "f32", "f32"), (90, 129, 257, 6, "f32", "f16"),
    (90, 257, 129, 13, "f32", "bf16"), (2600, 1100, 700, 16, "f32", "f32"), (200, 11008, 300, 16, "f16", "f16"), (4100, 5000, 4096, 8, "f16", "f16"),
]


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", ONE_TOKEN_EDGES)
def test_one_token_calls_are_fp32(gpu, m, n, k, l, env_dtype, x_dtype):
    """Products of envelope entries, signs and activations in fp32, sums of at most a few dozen per lane, then over lanes,
    waves and workgroups: the gate of the fp32 path.  The second layer's products of two envelope entries lie outside
    the range of fp32 (its What is the first one's)."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 1, seed=9 + m, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    Xd = _to_dev(torch, X, x_dtype)
    got = mb.mdbf_forward(mb.DeviceLayer.from_host(L), Xd, y_dtype="f32")
    assert orc.max_rel_error(got.cpu().numpy(), ref) <= 2e-5
    assert torch.equal(got, mb.mdbf_forward(mb.DeviceLayer.from_host(L), Xd, y_dtype="f32"))
    if env_dtype != "f16":
        H = dict(L, A=L["A"] * np.float32(2.0 ** 70), Q=L["Q"] * np.float32(2.0 ** 70), G=L["G"] * np.float32(2.0 ** -70), B=L["B"] * np.float32(2.0 ** -30))
        got = mb.mdbf_forward(mb.DeviceLayer.from_host(H), Xd, y_dtype="f32").cpu().numpy() * 2.0 ** -40
        assert orc.max_rel_error(got, ref) <= 2e-5


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype,y_dtype", [
    (16, 128, 16000, 16, "f32", "f32", "f32"), (17, 130, 9100, 5, "bf16", "f16", "f32"), (1000, 129, 8001, 8, "f16", "bf16", "f16"),
    (2000, 72, 8009, 3, "f32", "f32", "f32"), (40, 11008, 2700, 16, "f32", "f16", "bf16"), (1, 1, 30000, 1, "f16", "f32", "f32"),
])
def test_one_token_calls_of_few_rows_and_long_contractions(gpu, m, n, k, l, env_dtype, x_dtype, y_dtype):
    """The second factor's blocks on two to eight workgroups per row tile, the last with fewer, beside a first factor that is
    split as well and others that are not; the sums are added in a launch of their own, which accumulates and converts; a
    graph's replays; nothing is written behind the workspace."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 1, seed=9 + m, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, x_dtype)
    size = mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32"), 1)
    ws = torch.full((size + 4096,), 77, dtype=torch.uint8, device="cuda:0")
    got = mb.mdbf_forward(dl, Xd, y_dtype="f32", workspace=ws[:size])
    assert orc.max_rel_error(got.cpu().numpy(), ref) <= 2e-5
    assert (ws[size:] == 77).all()
    assert torch.equal(mb.mdbf_forward(dl, Xd, y_dtype="f32", Y=got.clone(), accumulate=True), got + got)
    out = mb.mdbf_forward(dl, Xd, y_dtype=y_dtype, workspace=ws[:size])
    assert torch.equal(out, got.to(out.dtype))
    Y = torch.empty_like(got)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mb.mdbf_forward(dl, Xd, y_dtype="f32", Y=Y, workspace=ws[:size])
    for _ in range(3):
        Y.fill_(-1.0)
        ws[:size].fill_(255)                             # (NaNs where partial sums will be)
        graph.replay()
        assert torch.equal(Y, got)


def test_one_token_call_of_more_threads_than_a_grid_dimension_holds(gpu):
    """8.4 million row tiles on eight waves each: the last tiles' rows are those of a layer that has them alone."""
    torch, mb = gpu
    n, k, rows = 64, 640, 64 * 16
    m = 2 ** 27 + rows                                   # (whole groups of 64 row tiles, stored one after the other)
    g = torch.Generator(device="cuda:0").manual_seed(1)
    words = lambda r, c: torch.randint(-2 ** 31, 2 ** 31 - 1, (mb.mdbf_packed_bytes(r, c) // 4,), dtype=torch.int32, generator=g, device="cuda:0")
    env = lambda r: torch.rand((r, 8), generator=g, device="cuda:0").to(torch.float16)
    SA, SB, A, Q, G, B = words(m, k), words(k, n), env(m), env(k), env(k), env(n)
    X = torch.randn((1, n), generator=g, device="cuda:0").to(torch.float16)
    Y = mb.mdbf_forward(mb.DeviceLayer(m, n, k, 8, SA, SB, A, Q, G, B), X, y_dtype="f16")
    part = mb.mdbf_packed_bytes(rows, k) // 4
    for t0, r0 in ((-part, m - rows), (0, 0)):
        end = mb.DeviceLayer(rows, n, k, 8, SA[t0:][:part], SB, A[r0:][:rows], Q, G, B)
        assert torch.equal(Y[:, r0:][:, :rows], mb.mdbf_forward(end, X, y_dtype="f16"))


@pytest.mark.parametrize("where", ["single", "plan"])
@pytest.mark.parametrize("l", [1, 4, 8, 13, 16])
@pytest.mark.parametrize("env_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("ein,eout,x", [(127, -110, -100), (127, 0, -100), (-125, 100, 100), (-123, 0, 100)])
def test_one_token_calls_with_envelopes_near_the_ends_of_fp32(gpu, ein, eout, x, env_dtype, l, where):
    """Entries of one factor's input side in [2^ein, 2^(ein + 1)), of its output side in [2^eout, 2^(eout + 1)): sums of
    their products leave fp32, or its normal range, although every entry times its activation and every result is in it.
    At the lower end an entry of the rebuilt factor is rounded at 2^-150, 2^-18 of it at most."""
    torch, mb = gpu
    m, n, k = 40, 300, 150
    L = synth.make_layer(m, n, k, l, seed=l, env_dtype="f32", env_kind="unit", signed_env=True)
    for f in "AQGB":
        L[f] = synth.round_to_dtype(np.sign(L[f]) * (1.0 + np.abs(L[f]) % 0.98), env_dtype)
    X = synth.make_activations(n, 1, seed=3, x_dtype="f32")
    ref = orc.forward_factored(*_oracle_args(L), X)
    Xd = _to_dev(torch, X * np.float32(2.0 ** x), "f32")
    for inner, outer in (("B", "G"), ("Q", "A")):
        H = dict(L, env_dtype=env_dtype)
        H[inner] = L[inner] * np.float32(2.0 ** ein)
        H[outer] = L[outer] * np.float32(2.0 ** eout)
        dl, Y = mb.DeviceLayer.from_host(H), torch.zeros((1, m), device="cuda:0")
        if where == "single":
            mb.mdbf_forward(dl, Xd, Y=Y)
        else:
            mb.BatchPlan([dl], [Xd], [Y]).run()
        assert orc.max_rel_error(Y.cpu().numpy().astype(np.float64) * 2.0 ** -(ein + eout + x), ref) <= 2e-5


@pytest.mark.parametrize("where", ["single", "forced", "plan"])
@pytest.mark.parametrize("l,T", [(8, 1), (16, 1), (16, 3)])
def test_non_finite_input_reaches_every_output_of_the_block_scaled_kernels(gpu, l, T, where):
    """The fp6 limbs saturate, the column sums carry infinities and NaNs: a bad value in any column of a block (each of
    the four operand registers of a lane holds other columns), in the input or in either factor's input-side envelope,
    leaves no output of its token finite, and the other tokens' alone."""
    torch, mb = gpu
    m, n, k = 150, 300, 260
    L = synth.make_layer(m, n, k, l, seed=l, env_dtype="f16", env_kind="llama", signed_env=True)
    dl = mb.DeviceLayer.from_host(L)
    X = torch.from_numpy(synth.make_activations(n, T, seed=7, x_dtype="f16")).half().cuda()
    Y = torch.zeros((T, m), dtype=torch.float32, device="cuda:0")
    plan = mb.BatchPlan([dl], [X], [Y], block_scaled=True)
    assert plan.kernel(1) == plan.kernel(2) == "stage_mx_kernel"

    def out():
        if where == "plan":
            plan.run()
            return Y
        return mb.mdbf_forward(dl, X, y_dtype="f32", block_scaled=where == "forced")
    ref = out().clone()
    assert torch.isfinite(ref).all()
    for t, rows in ((X[T - 1], n), (dl.B[:, l - 1], n), (dl.Q[:, 0], k)):
        for c in list(range(128)) + [rows - 1]:
            for bad in (float("inf"), float("nan")):
                keep = t[c].clone()
                t[c] = bad
                got = out()
                assert not torch.isfinite(got[T - 1]).any(), (rows, c, bad)
                if rows == n and t.data_ptr() == X[T - 1].data_ptr():
                    assert torch.equal(got[:T - 1], ref[:T - 1])
                t[c] = keep
    assert torch.equal(out(), ref)


# ---------------------------------------------------------------- many layers in one launch pair
def _batch_case(gpu, specs, tokens=lambda i: 1 + (i % 2)):
    torch, mb = gpu
    layers, Xs, Ys, singles, refs = [], [], [], [], []
    for i, (m, n, k, l) in enumerate(specs):
        L = synth.make_layer(m, n, k, l, seed=400 + i, env_dtype="f16", env_kind="llama")
        X = synth.make_activations(n, tokens(i), seed=500 + i, x_dtype="f16")
        dl = mb.DeviceLayer.from_host(L)
        Xd = _to_dev(torch, X, "f16")
        layers.append(dl)
        Xs.append(Xd)
        Ys.append(torch.zeros((Xd.shape[0], m), dtype=torch.float32, device="cuda:0"))
        singles.append(mb.mdbf_forward(dl, Xd))
        refs.append(orc.forward_factored(*_oracle_args(L), X))
    plan = mb.BatchPlan(layers, Xs, Ys)
    plan.run()
    torch.cuda.synchronize()
    return Ys, singles, refs


def test_batch_mixed_layers(gpu):
    """Layers of different shapes and envelope ranks in one plan (served by the general kernel)."""
    specs = [(256, 256, 128, 4), (530, 2100, 1100, 16), (100, 1030, 200, 8), (4096, 4096, 2656, 16)]
    Ys, singles, refs = _batch_case(gpu, specs)
    for Yb, Y1, ref in zip(Ys, singles, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL
        assert orc.max_rel_error(Y1.cpu().numpy(), ref) <= TOL
        # the kernel variants quantise the staged activations differently (fp16 vs three fp6 limbs)
        assert orc.max_rel_error(Yb.cpu().numpy(), Y1.cpu().numpy().astype(np.float64)) <= 5e-4


def test_batch_fast_layers_equal_single_calls(gpu):
    """All layers l = 16 / fp16, one token.  A plan this small runs the fp16-staged kernel, the single calls the
    block-scaled one with the contraction split across workgroups: the two quantise the staged activations
    differently (fp16 against three fp6 limbs)."""
    torch, mb = gpu
    specs = [(530, 2104, 1104, 16), (4096, 4096, 2656, 16), (272, 1032, 4096, 16), (4096, 4096, 2656, 16)]
    Ys, singles, refs = _batch_case(gpu, specs, tokens=lambda i: 1)
    for Yb, Y1, ref in zip(Ys, singles, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL
        assert orc.max_rel_error(Yb.cpu().numpy(), Y1.cpu().numpy().astype(np.float64)) <= 5e-4


def test_plan_of_several_tokens_equals_single_calls(gpu):
    """From a few tokens on, plans and single calls both take the reconstruct-order variant: the same
    fp16-rounded factors and activations; a short single call adds its column blocks in four partial sums
    (split over the waves of a workgroup), a plan in one run, so the fp32 results agree to rounding."""
    torch, mb = gpu
    specs = [(530, 2104, 1104, 16), (272, 1032, 4096, 16), (96, 200, 150, 5), (4096, 4096, 2656, 16)]
    Ys, singles, refs = _batch_case(gpu, specs, tokens=lambda i: 4 + 3 * i)
    for Yb, Y1, ref in zip(Ys, singles, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL
        assert orc.max_rel_error(Yb.cpu().numpy(), Y1.cpu().numpy().astype(np.float64)) <= 2e-5


# ---------------------------------------------------------------- prefill-shaped batch of tokens
@pytest.mark.parametrize("x_dtype", ["f16", "bf16"])
def test_prefill_tokens_sampled_against_oracle(gpu, x_dtype):
    """4096x4096, k=2656, l=16, 2048 tokens, envelopes |N|+0.1 (outputs reach 1e6: fp32 Y).
    All 2048 rows are computed on the GPU; 6 sampled tokens are checked against the oracle."""
    torch, mb = gpu
    L, X = synth.config_prefill(T=2048, x_dtype=x_dtype)
    dl = mb.DeviceLayer.from_host(L)
    Xd = _to_dev(torch, X, x_dtype)
    Y = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    torch.cuda.synchronize()
    Yh = Y.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(Yh))
    rows = [0, 1, 777, 1024, 2046, 2047]
    ref = orc.forward_factored(*_oracle_args(L), X[rows])
    assert orc.max_rel_error(Yh[rows], ref) <= TOL
    # every token is an independent product: rows must not leak into each other
    Ysub = mb.mdbf_forward(dl, Xd[760:800].contiguous(), y_dtype="f32")
    torch.cuda.synchronize()
    assert torch.equal(Ysub, Y[760:800])
    # a single token takes the small-batch kernel variant, which quantises the activations differently
    Y1 = mb.mdbf_forward(dl, Xd[777:778].contiguous(), y_dtype="f32")
    torch.cuda.synchronize()
    assert orc.max_rel_error(Y1[0].cpu().numpy(), Yh[777]) <= 5e-4


# ---------------------------------------------------------------- many tokens: the reconstruct-order variant
MANY = [
    # m, n, k, l, T, env_dtype, x_dtype: every token-slab count, ragged shapes, all envelope ranks and dtypes
    (16, 128, 16, 16, 17, "f16", "f16"),
    (40, 300, 70, 3, 33, "f32", "f32"),
    (130, 129, 257, 8, 65, "bf16", "bf16"),
    (530, 2100, 1100, 16, 100, "f16", "f16"),
    (100, 1030, 200, 1, 130, "f16", "f32"),
    (1100, 520, 2105, 16, 300, "f16", "bf16"),
    (530, 2100, 1100, 8, 100, "f16", "f16"),
    (1100, 520, 2104, 8, 40, "f16", "bf16"),
]


@pytest.mark.parametrize("m,n,k,l,T,env_dtype,x_dtype", MANY)
def test_many_token_variant(gpu, m, n, k, l, T, env_dtype, x_dtype):
    L = synth.make_layer(m, n, k, l, seed=7 * m + n + k, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=55 + T, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, x_dtype, "f32")
    assert orc.max_rel_error(got, ref) <= TOL


def test_many_token_exact_integer_inputs(gpu):
    """All-ones envelopes (l = 4) and x in {-1,0,1}, 50 tokens: the rebuilt factor is +-l, every partial sum
    is an integer below 2^11 in stage 1's fp16 operands and below 2^24 in fp32: bit for bit."""
    m, n, k, l, T = 200, 520, 96, 4, 50
    L = synth.make_layer(m, n, k, l, seed=61, env_dtype="f16", env_kind="ones")
    X = synth.make_activations(n, T, seed=62, x_dtype="f16", kind="ternary")
    ref = orc.forward_factored(*_oracle_args(L), X)
    # stage 2 feeds z = l * P1 through fp16: exact while |z| < 2048
    _, Z = orc.forward_factored(*_oracle_args(L), X, return_intermediates=True)
    got = _run(gpu, L, X, "f16", "f32")
    if np.max(np.abs(Z)) < 2048:
        np.testing.assert_array_equal(got, ref)
    else:
        assert orc.max_rel_error(got, ref) <= TOL


def test_many_token_batch(gpu):
    torch, mb = gpu
    specs = [(530, 2104, 1104, 16, 40), (272, 1032, 4096, 16, 17), (96, 200, 150, 5, 64)]
    layers, Xs, Ys, refs = [], [], [], []
    for i, (m, n, k, l, T) in enumerate(specs):
        L = synth.make_layer(m, n, k, l, seed=500 + i, env_dtype="f16", env_kind="llama", signed_env=True)
        X = synth.make_activations(n, T, seed=600 + i, x_dtype="f16")
        layers.append(mb.DeviceLayer.from_host(L))
        Xs.append(_to_dev(torch, X, "f16"))
        Ys.append(torch.zeros((T, m), dtype=torch.float32, device="cuda:0"))
        refs.append(orc.forward_factored(*_oracle_args(L), X))
    plan = mb.BatchPlan(layers, Xs, Ys)
    plan.run()
    torch.cuda.synchronize()
    for Yb, ref in zip(Ys, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL


# ---------------------------------------------------------------- residual stacks: Y += What x
@pytest.mark.parametrize("T,y_dtype,variant", [(1, "f32", "auto"), (1, "f16", "auto"), (1, "f32", "block_scaled"),
                                               (1, "f32", "precise"), (6, "f32", "auto"), (40, "bf16", "auto"),
                                               (1, "f32", "generic")])
def test_residual_stack_accumulates(gpu, T, y_dtype, variant):
    """Two independently factorised terms applied to the same Y, the second with MDBF_FLAG_ACCUMULATE."""
    torch, mb = gpu
    m, n = 530, 2104
    l = 5 if variant == "generic" else 16
    terms = [synth.make_layer(m, n, k, l, seed=900 + i, env_dtype="f16", env_kind="llama", signed_env=True)
             for i, k in enumerate((1104, 520))]
    X = synth.make_activations(n, T, seed=910, x_dtype="f16")
    ref = orc.forward_residual_stack([_oracle_args(L) for L in terms], X)
    Xd = _to_dev(torch, X, "f16")
    kw = dict(precise=(variant == "precise"), block_scaled=(variant == "block_scaled"))
    Y = mb.mdbf_forward(mb.DeviceLayer.from_host(terms[0]), Xd, y_dtype=y_dtype, **kw)
    mb.mdbf_forward(mb.DeviceLayer.from_host(terms[1]), Xd, y_dtype=y_dtype, Y=Y, accumulate=True, **kw)
    torch.cuda.synchronize()
    slack = {"f32": 0.0, "f16": 2.0 ** -10, "bf16": 2.0 ** -7}[y_dtype]   # two roundings to the output type
    assert orc.max_rel_error(Y.float().cpu().numpy(), ref) <= TOL + slack


def test_residual_stack_in_a_plan(gpu):
    torch, mb = gpu
    m, n = 272, 1032
    terms = [synth.make_layer(m, n, k, 16, seed=920 + i, env_dtype="f16", env_kind="llama") for i, k in enumerate((4096, 1104))]
    X = synth.make_activations(n, 1, seed=930, x_dtype="f16")
    ref = orc.forward_residual_stack([_oracle_args(L) for L in terms], X)
    Xd = _to_dev(torch, X, "f16")
    Y = torch.zeros((1, m), dtype=torch.float32, device="cuda:0")
    # the two terms of one output must not share a plan (their order is not defined inside one launch)
    for i, L in enumerate(terms):
        plan = mb.BatchPlan([mb.DeviceLayer.from_host(L)], [Xd], [Y], accumulate=(i > 0))
        plan.run()
    torch.cuda.synchronize()
    assert orc.max_rel_error(Y.cpu().numpy(), ref) <= TOL


PLAN_FORMS = [
    # copies of the layers, tokens: 2, 4, 8 and 16 row tiles per item, one to four runs over the contraction, each slab count
    (1, 16), (1, 9), (1, 32), (1, 64), (8, 5), (8, 17), (8, 33), (16, 16), (45, 4), (45, 40), (50, 8), (260, 6), (260, 9),
]


@pytest.mark.parametrize("copies,T", PLAN_FORMS)
@pytest.mark.parametrize("l,x_dtype", [(16, "f16"), (8, "bf16"), (5, "f32")])
def test_item_forms_of_many_token_plans(gpu, copies, T, l, x_dtype):
    """Contractions of one block (three of four runs are empty), five and nine; row tiles that do not fill the last
    item.  Against the oracle at the fp16 gate, copies among each other bit for bit."""
    torch, mb = gpu
    layers, Xs, Ys, refs = [], [], [], []
    for i, (m, n, k) in enumerate([(2100, 72, 600), (52, 1100, 120)]):
        L = synth.make_layer(m, n, k, l, seed=40 + i, env_dtype="f16", env_kind="unit", signed_env=True)
        X = synth.make_activations(n, T, seed=50 + i, x_dtype=x_dtype)
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, x_dtype)
        layers += [dl] * copies
        Xs += [Xd] * copies
        Ys.append(torch.zeros((copies, T, m), dtype=torch.float32, device="cuda:0"))
    plan = mb.BatchPlan(layers, Xs, [y for Y in Ys for y in Y])
    assert plan.kernel(1) == "stage_gemm_kernel" and plan.launches() == 2
    for _ in range(2):
        plan.run()
    for Y, ref in zip(Ys, refs):
        assert orc.max_rel_error(Y[0].cpu().numpy(), ref) <= TOL
        assert torch.equal(Y, Y[:1].expand_as(Y))


@pytest.mark.parametrize("copies,T", [(1, 8), (3, 16), (3, 32), (7, 6), (7, 40), (12, 13), (30, 7), (30, 20), (45, 5), (70, 8), (70, 12)])
@pytest.mark.parametrize("l", [4, 13])
def test_item_forms_of_many_token_plans_with_fp32_envelopes(gpu, copies, T, l):
    """Items of 4, 8 and 16 row tiles, one, two and four runs over contractions of 1, 5, 9 and 41 blocks, pairs of row tiles
    and single ones, all loaded element by element.  (Rounded to fp16 as the fp16 envelopes are.)"""
    torch, mb = gpu
    layers, Xs, Ys, refs = [], [], [], []
    for i, (m, n, k) in enumerate([(2100, 72, 600), (52, 1100, 120), (72, 600, 5200)]):
        L = synth.make_layer(m, n, k, l, seed=40 + i, env_dtype="f32", env_kind="unit", signed_env=True)
        X = synth.make_activations(n, T, seed=50 + i, x_dtype="f32")
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, "f32")
        layers += [dl] * copies
        Xs += [Xd] * copies
        Ys.append(torch.zeros((copies, T, m), dtype=torch.float32, device="cuda:0"))
    plan = mb.BatchPlan(layers, Xs, [y for Y in Ys for y in Y])
    assert plan.kernel(1) == "stage_gemm_kernel" and plan.launches() == 2
    for _ in range(2):
        plan.run()
    for Y, ref in zip(Ys, refs):
        assert orc.max_rel_error(Y[0].cpu().numpy(), ref) <= TOL
        assert torch.equal(Y, Y[:1].expand_as(Y))


@pytest.mark.parametrize("n,k,l,x_dtype", [(264, 136, 16, "f16"), (136, 264, 8, "bf16"), (264, 136, 16, "f32"), (131, 137, 5, "f16")])
def test_tile_shapes_of_long_calls(gpu, n, k, l, x_dtype):
    """256 row tiles with lengths that take each tile shape on the second factor (2 x 8, 2 x 6, 2 x 4, 2 x 2, 1 x 2), the last
    slabs cut, the last rows missing: the same bits as the longest call's, which meets the oracle; fp16 copies and operands
    as they are."""
    torch, mb = gpu
    m = 4090
    L = synth.make_layer(m, n, k, l, seed=n + k + l, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 2041, seed=7, x_dtype=x_dtype)
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, x_dtype)
    full = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    rows = list(range(0, 2041, 51)) + list(range(2009, 2041))
    assert orc.max_rel_error(full[rows].cpu().numpy(), orc.forward_factored(*_oracle_args(L), X[rows])) <= TOL
    for T in (65, 97, 290, 383, 639, 769, 1300, 2041):
        ws = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32", precise=True), T), dtype=torch.uint8, device="cuda:0")
        assert torch.equal(mb.mdbf_forward(dl, Xd[:T], y_dtype="f32"), full[:T]), T
        assert torch.equal(mb.mdbf_forward(dl, Xd[:T], y_dtype="f32", workspace=ws), full[:T]), T


@pytest.mark.parametrize("n,k,l,x_dtype", [(300, 520, 16, "f16"), (301, 515, 8, "bf16"), (130, 260, 5, "f32")])
def test_long_calls_of_seven_slabs_at_a_time(gpu, n, k, l, x_dtype):
    """512 row tiles in seven pieces of seven slabs, the last slab of one row, of four, and whole: the same bits as a longer
    call's, which meets the oracle; fp16 copies and operands as they are."""
    torch, mb = gpu
    L = synth.make_layer(8186, n, k, l, seed=n + k + l, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 1100, seed=8, x_dtype=x_dtype)
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, x_dtype)
    full = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    rows = list(range(0, 1100, 51)) + list(range(752, 784))
    assert orc.max_rel_error(full[rows].cpu().numpy(), orc.forward_factored(*_oracle_args(L), X[rows])) <= TOL
    for T in (769, 772, 784):
        ws = torch.empty(mb.mdbf_workspace_bytes(dl.desc(x_dtype, "f32", precise=True), T), dtype=torch.uint8, device="cuda:0")
        assert torch.equal(mb.mdbf_forward(dl, Xd[:T], y_dtype="f32"), full[:T]), T
        assert torch.equal(mb.mdbf_forward(dl, Xd[:T], y_dtype="f32", workspace=ws), full[:T]), T


@pytest.mark.parametrize("n,k", [(640, 4090), (1160, 4096), (1536, 1100), (1544, 8200)])
def test_bf16_calls_of_33_to_64_tokens(gpu, n, k):
    """Both sides of the length from which two row tiles share the conversion of bf16 activations, few and many row tiles:
    any length from 33 to 64 is the same bits as 64 tokens, which meet the oracle."""
    torch, mb = gpu
    L = synth.make_layer(72, n, k, 8, seed=n + k, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 64, seed=9, x_dtype="bf16")
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, "bf16")
    full = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    assert orc.max_rel_error(full.cpu().numpy(), orc.forward_factored(*_oracle_args(L), X)) <= TOL
    for T in (33, 47, 49, 63):
        assert torch.equal(mb.mdbf_forward(dl, Xd[:T], y_dtype="f32"), full[:T]), T


@pytest.mark.parametrize("m,k,copies,T", [(2100, 600, 50, 8), (2100, 600, 100, 5), (52, 300, 1500, 6)])
@pytest.mark.parametrize("l,x_dtype", [(16, "f16"), (8, "bf16"), (5, "f32")])
def test_rows_beyond_fp16_stay_by_themselves(gpu, m, k, copies, T, l, x_dtype):
    """Plans that take two row tiles in one product (items of 8 and 16 tiles, one and two runs): a row whose entries leave
    fp16 and one of NaNs are not finite, the other rows the same bits as without them; results are added once."""
    torch, mb = gpu
    L = synth.make_layer(m, 72, k, l, seed=60, env_dtype="f16", env_kind="unit", signed_env=True)
    L["Q"][:, 0] = 2.0                                      # row 5 of A: every entry of its E beyond fp16
    bad = dict(L, A=L["A"].copy())
    bad["A"][5], bad["A"][5, 0], bad["A"][m - 1, l - 1] = 0.0, 60000.0, np.nan
    X = synth.make_activations(72, T, seed=61, x_dtype=x_dtype)
    outs = []
    for which in (L, bad):
        dl, Xd = mb.DeviceLayer.from_host(which), _to_dev(torch, X, x_dtype)
        Y = torch.ones((copies, T, m), dtype=torch.float32, device="cuda:0")
        plan = mb.BatchPlan([dl] * copies, [Xd] * copies, list(Y), accumulate=True)
        assert plan.kernel(2) == "stage_gemm_kernel"
        plan.run()
        outs.append(Y)
    clean, got = outs
    ref = orc.forward_factored(*_oracle_args(L), X)
    assert orc.max_rel_error(clean[0].cpu().numpy() - 1.0, ref) <= TOL + 2.0 ** -23 / np.abs(ref).max()
    assert not torch.isfinite(got[:, :, [5, m - 1]]).any()
    keep = [r for r in range(m) if r not in (5, m - 1)]
    assert torch.equal(got[:, :, keep], clean[:, :, keep])


@pytest.mark.parametrize("tokens", [(1, 1, 1), (3, 3, 3), (1, 9, 2)])
@pytest.mark.parametrize("x_dtype,y_dtype", [("f16", "f32"), ("f32", "f16")])
def test_small_plans_of_rank_16(gpu, tokens, x_dtype, y_dtype):
    """Items of four row tiles, each wave an eighth of the contraction: one block per wave, two (the last waves have one or
    none), eleven in three chunks of their own scale; a last item of one, two and three tiles; the second pass adds."""
    torch, mb = gpu
    layers, Xs, Ys, refs = [], [], [], []
    for i, ((m, n, k), T) in enumerate(zip([(530, 1024, 1160), (16, 1160, 2050 // 8 * 8), (176, 11008, 1040)], tokens)):
        L = synth.make_layer(m, n, k, 16, seed=70 + i, env_dtype="f16", env_kind="llama", signed_env=True)
        X = synth.make_activations(n, T, seed=80 + i, x_dtype=x_dtype)
        X[:, : n // 2] *= 2.0 ** -9                       # chunks of other magnitudes
        X = synth.round_to_dtype(X, x_dtype)
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        layers.append(mb.DeviceLayer.from_host(L))
        Xs.append(_to_dev(torch, X, x_dtype))
        Ys.append(torch.zeros((T, m), dtype=torch.float32 if y_dtype == "f32" else torch.float16, device="cuda:0"))
    plan = mb.BatchPlan(layers, Xs, Ys, accumulate=True)
    assert plan.kernel(1) == plan.kernel(2) == "stage_fast_kernel" and plan.launches() == 4
    for passes in (1, 2):
        plan.run()
        for Y, ref in zip(Ys, refs):
            assert orc.max_rel_error(Y.float().cpu().numpy(), passes * ref) <= TOL + (2.0 ** -10 if y_dtype == "f16" else 0.0)


@pytest.mark.parametrize("k", [1024, 1152, 1288, 1808])
def test_small_plans_of_rank_16_with_an_infinite_envelope_entry(gpu, k):
    """8, 9, 11 and 15 blocks on eight waves, some of which have none: terms of one sign times an infinity are one."""
    torch, mb = gpu
    L = synth.make_layer(40, 1024, k, 16, seed=k, env_dtype="f16", env_kind="unit")
    L["SA"], L["SB"] = np.abs(L["SA"]), np.abs(L["SB"])
    X = np.abs(synth.make_activations(1024, 1, seed=1, x_dtype="f16")) * np.float32(2.0 ** -6)
    Xd, outs = _to_dev(torch, X, "f16"), []
    for value in (1.0, np.inf):
        L["A"][5, 3] = value
        Y = torch.zeros((1, 40), dtype=torch.float32, device="cuda:0")
        plan = mb.BatchPlan([mb.DeviceLayer.from_host(L)], [Xd], [Y])
        assert plan.kernel(2) == "stage_fast_kernel"
        plan.run()
        outs.append(Y[0])
    clean, got = outs
    assert torch.isfinite(clean).all() and got[5] == float("inf")
    assert torch.equal(torch.cat((got[:5], got[6:])), torch.cat((clean[:5], clean[6:])))


PAIR_EDGES = [
    # m, n, k, l, env, x: as many pieces of the first factor (16 x 128) as one launch takes of each kind of rows, and more; one,
    # two and three blocks of the second one, its last row tile on a second slot; sizes that are no multiples of anything
    (256, 256, 128, 4, "f32", "f32"), (33, 640, 64, 4, "f32", "bf16"), (33, 641, 64, 4, "f32", "f32"), (47, 383, 61, 8, "f32", "f16"),
    (300, 384, 128, 16, "f16", "f16"), (300, 385, 128, 16, "f16", "f16"), (520, 127, 384, 16, "f16", "f32"), (4099, 101, 383, 8, "f16", "bf16"),
    (8190, 101, 383, 8, "f16", "f16"), (50, 255, 63, 3, "f16", "f16"), (50, 129, 64, 16, "bf16", "bf16"), (17, 1000, 15, 11, "f32", "f32"),
    (1, 1, 1, 1, "f16", "f16"), (4, 4, 4, 4, "f32", "f32"), (19, 5, 130, 4, "f32", "f32"), (70, 1030, 520, 4, "f32", "f32"),
    # more than 256 row tiles of one and two blocks on the slots of 256 workgroups (two, three and all eight of them, three of four),
    # and of three blocks past what 256 workgroups take (8192 rows: the two sides of that line)
    (4113, 130, 128, 16, "f16", "f16"), (11008, 130, 100, 8, "f16", "f16"), (32767, 65, 90, 4, "f32", "f32"), (8200, 101, 250, 16, "f16", "f16"),
    (8192, 101, 383, 8, "f16", "f16"), (8200, 101, 383, 8, "f16", "f16"),
]


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", PAIR_EDGES)
def test_small_one_token_calls(gpu, m, n, k, l, env_dtype, x_dtype):
    """Both factors in one launch, z in LDS, and layers just too large for it: the gate of the fp32 path; a second call adds;
    an infinity in one row of the last envelope stays in that row's output; the scratch array's entry point has the same bits."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    X = synth.make_activations(n, 1, seed=9 + m, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, x_dtype)
    got = mb.mdbf_forward(_between_nans(torch, dl), Xd, y_dtype="f32")
    assert orc.max_rel_error(got.cpu().numpy(), ref) <= 2e-5
    assert torch.equal(mb.mdbf_forward(dl, Xd, y_dtype="f32", Y=got.clone(), accumulate=True), got + got)
    out = torch.zeros((1, m), dtype=torch.float32, device="cuda:0")
    assert torch.equal(mb.mdbf_forward_static(dl, Xd, out), got)
    dl.A[m - 1, l - 1] = float("inf")
    again = mb.mdbf_forward(dl, Xd, y_dtype="f32")
    assert not torch.isfinite(again[0, m - 1]) and torch.equal(again[0, :m - 1], got[0, :m - 1])


@pytest.mark.parametrize("m,n,k,l,env_dtype,dtype", [(256, 256, 128, 4, "f32", "f32"), (256, 256, 128, 16, "f16", "f16"), (300, 384, 100, 8, "f16", "bf16"),
                                                     (4096, 127, 60, 16, "f16", "f32"), (4096, 4096, 300, 16, "f16", "f16")])
def test_one_token_calls_in_place(gpu, m, n, k, l, env_dtype, dtype):
    """Y over X: the same memory, and 16 bytes behind its start; overwritten, and added to itself.  Both places have the same bits,
    those of two launches, which meet the oracle at the gate of the fp32 path and the rounding of a 16-bit Y (2^-11, 2^-8; of the
    product and of the sum where it is added)."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="llama", signed_env=True)
    X = synth.make_activations(n, 1, seed=3, x_dtype=dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    dl, Xd = mb.DeviceLayer.from_host(L), _to_dev(torch, X, dtype)
    unit = {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype]
    shift = 16 // Xd.element_size()

    def in_place(offset, accumulate):
        buf = torch.zeros(offset + max(m, n), dtype=Xd.dtype, device="cuda:0")
        buf[:n] = Xd[0]
        before = buf[offset:offset + m].float().cpu().numpy().astype(np.float64)
        Y = buf[offset:offset + m].unsqueeze(0)
        mb.mdbf_forward(dl, buf[:n].unsqueeze(0), y_dtype=dtype, Y=Y, accumulate=accumulate)
        return Y, before if accumulate else 0.0

    for accumulate in (False, True):
        for offset in (0, shift):
            Y, before = in_place(offset, accumulate)
            assert orc.max_rel_error(Y.float().cpu().numpy(), ref + before) <= 2e-5 + (2 if accumulate else 1) * unit, (offset, accumulate)
    assert torch.equal(in_place(0, False)[0], in_place(shift, False)[0])


ONE_PLANS = [
    # specs (m, n, k, l), envelopes, activations, tokens: ranks of every class and mixed ones, odd row pitches, contractions of
    # one block and of more than one per wave, row tiles that do not fill the last item
    ([(530, 2101, 1107, 8), (16, 100, 40, 8)], "f16", "f16", 3), ([(300, 257, 2100, 3), (130, 129, 5, 3)], "bf16", "bf16", 2),
    ([(260, 300, 130, 4), (200, 1030, 515, 2)], "f32", "f32", 3), ([(256, 256, 128, 4), (530, 2100, 1100, 16), (100, 1030, 200, 8)], "f16", "bf16", 1),
    ([(90, 700, 650, 16), (33, 1, 3, 1)], "f32", "f16", 2), ([(40, 131, 200, 15), (40, 131, 200, 9)], "bf16", "f32", 3),
]


@pytest.mark.parametrize("specs,env_dtype,x_dtype,T", ONE_PLANS)
def test_plans_of_few_tokens_in_fp32(gpu, specs, env_dtype, x_dtype, T):
    """Plans that neither the fp16-staged nor (at their size) the block-scaled kernel serves: the arithmetic of single
    one-token calls, the gate of the fp32 path; an infinity stays in its layer and token."""
    torch, mb = gpu
    layers, Xs, Ys, refs = [], [], [], []
    for i, (m, n, k, l) in enumerate(specs):
        L = synth.make_layer(m, n, k, l, seed=70 + i, env_dtype=env_dtype, env_kind="unit", signed_env=True)
        X = synth.make_activations(n, T, seed=80 + i, x_dtype=x_dtype)
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        layers.append(mb.DeviceLayer.from_host(L))
        Xs.append(_to_dev(torch, X, x_dtype))
        Ys.append(torch.zeros((T, m + 3), dtype=torch.float32, device="cuda:0")[:, :m])
    plan = mb.BatchPlan(layers, Xs, Ys)
    assert plan.kernel(1) == plan.kernel(2) == "stage_one_kernel" and plan.launches() == 2
    plan.run()
    for Y, ref in zip(Ys, refs):
        assert orc.max_rel_error(Y.cpu().numpy(), ref) <= 2e-5
    first = [Y.clone() for Y in Ys]
    Xs[0][T - 1, -1] = float("inf")
    plan.run()
    assert not torch.isfinite(Ys[0][T - 1]).any() and torch.equal(Ys[0][:T - 1], first[0][:T - 1])
    for Y, before in zip(Ys[1:], first[1:]):
        assert torch.equal(Y, before)


def _between_nans(torch, dl):
    """The layer with every envelope factor a 16-byte aligned view into a buffer of NaNs."""
    def view(e):
        buf = torch.full((16 + e.numel() + 16,), float("nan"), dtype=e.dtype, device=e.device)
        v = buf[16:16 + e.numel()].view(e.shape)
        v.copy_(e)
        return v
    return type(dl)(dl.m, dl.n, dl.k, dl.l, dl.SA_packed, dl.SB_packed, *[view(e) for e in (dl.A, dl.Q, dl.G, dl.B)])


@pytest.mark.parametrize("m,n,k,l,env_dtype,x_dtype", ONE_TOKEN_EDGES)
def test_one_token_calls_use_nothing_behind_the_envelopes(gpu, m, n, k, l, env_dtype, x_dtype):
    """The last rows' vectors end with the factor: what lies behind it meets zero modes only, and a NaN there would stay one."""
    torch, mb = gpu
    L = synth.make_layer(m, n, k, l, seed=m + n + k + l, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    Xd = _to_dev(torch, synth.make_activations(n, 1, seed=9 + m, x_dtype=x_dtype), x_dtype)
    dl = mb.DeviceLayer.from_host(L)
    assert torch.equal(mb.mdbf_forward(_between_nans(torch, dl), Xd), mb.mdbf_forward(dl, Xd))


@pytest.mark.parametrize("env_dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("m,n,k,l", [(33, 1, 3, 1), (17, 3, 1, 1), (20, 2, 2, 1), (18, 1, 1, 2), (40, 1, 2, 3), (5, 4, 1, 1), (9, 7, 1, 1)])
def test_plans_of_mixed_ranks_with_the_smallest_factors(gpu, m, n, k, l, env_dtype):
    """Rows of 16 modes at most next to a factor of fewer entries than a lane's vector holds (four in fp32, eight in the
    16-bit types)."""
    torch, mb = gpu
    specs = [(90, 700, 650, 16), (m, n, k, l)]
    layers, Xs, Ys, refs = [], [], [], []
    for i, s in enumerate(specs):
        L = synth.make_layer(*s, seed=70 + i, env_dtype=env_dtype, env_kind="unit", signed_env=True)
        X = synth.make_activations(s[1], 2, seed=80 + i, x_dtype="f32")
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        layers.append(_between_nans(torch, mb.DeviceLayer.from_host(L)))
        Xs.append(_to_dev(torch, X, "f32"))
        Ys.append(torch.zeros((2, s[0]), dtype=torch.float32, device="cuda:0"))
    plan = mb.BatchPlan(layers, Xs, Ys)
    assert plan.kernel(1) == plan.kernel(2) == "stage_one_kernel"
    plan.run()
    for Y, ref in zip(Ys, refs):
        assert orc.max_rel_error(Y.cpu().numpy(), ref) <= 2e-5


# ---------------------------------------------------------------- the synthetic decoder stack
@pytest.mark.parametrize("budget", ["1.0", "1.5", "2.0"])
@pytest.mark.parametrize("T", [1, 8])
def test_decoder_stack_layer_through_batch(gpu, budget, T):
    """One layer of the 32-layer stack (q,k,v,o,gate,up,down: 7 independent products) per budget,
    issued as one plan; each matrix is compared with the oracle."""
    torch, mb = gpu
    layer_idx = {"1.0": 0, "1.5": 15, "2.0": 31}[budget]
    layers, Xs, Ys, refs = [], [], [], []
    for mat in range(7):
        L, X = synth.stack_matrix(budget, layer_idx, mat, T=T)
        layers.append(mb.DeviceLayer.from_host(L))
        Xs.append(_to_dev(torch, X, "f16"))
        Ys.append(torch.zeros((T, L["m"]), dtype=torch.float32, device="cuda:0"))
        refs.append(orc.forward_factored(*_oracle_args(L), X))
        sp = synth.stack_matrix_spec(budget, layer_idx, mat)
        assert abs(mb.mdbf_bpw(sp["m"], sp["n"], sp["k"], sp["l"]) - float(budget)) < 0.01
    plan = mb.BatchPlan(layers, Xs, Ys)
    plan.run()
    torch.cuda.synchronize()
    for Yb, ref in zip(Ys, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL


def test_block_scaled_plan_with_more_items_than_workgroups(gpu):
    """300 small problems of mixed contraction lengths in one block-scaled plan: more work items than the
    device holds workgroups, so that the host's cost-balanced item order and the kernel's walk over several
    items per workgroup are both on the path; every problem is compared with the oracle."""
    torch, mb = gpu
    rng = np.random.default_rng(31)
    layers, Xs, Ys, refs = [], [], [], []
    for i in range(300):
        m = int(rng.integers(17, 80))
        n = int(rng.choice([256, 300, 640, 1280]))
        k = int(rng.choice([130, 256, 640]))
        L = synth.make_layer(m, n, k, 16, seed=7000 + i, env_dtype="f16", env_kind="llama", signed_env=True)
        X = synth.make_activations(n, 1, seed=8000 + i, x_dtype="f16")
        layers.append(mb.DeviceLayer.from_host(L))
        Xs.append(_to_dev(torch, X, "f16"))
        Ys.append(torch.zeros((1, m), dtype=torch.float32, device="cuda:0"))
        refs.append(orc.forward_factored(*_oracle_args(L), X))
    plan = mb.BatchPlan(layers, Xs, Ys, block_scaled=True)
    for _ in range(2):                      # the plan is reusable
        plan.run()
    torch.cuda.synchronize()
    for Yb, ref in zip(Ys, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL


# ---------------------------------------------------------------- factors with the structure of a quantisation run
@pytest.mark.parametrize("rows,cols,R,l,outer", [(320, 288, 96, 4, 1), (272, 400, 160, 16, 0), (272, 400, 160, 16, 2)])
@pytest.mark.parametrize("variant", ["auto", "block_scaled", "tokens", "precise"])
def test_quantized_structured_factors(gpu, rows, cols, R, l, outer, variant):
    """The layer comes from the quantizer oracle run on a dense matrix with a decaying spectrum: sign masks
    correlated with the weights, envelope modes of mixed sign and falling size (the i.i.d. factors of the
    benchmark configurations have neither)."""
    from oracle import mdbf_quantizer as qz
    if variant == "block_scaled" and l != 16:
        pytest.skip("the block-scaled kernel takes rank-16 envelopes")
    W = synth.structured_weight(rows, cols, seed=rows + cols + l)
    L = qz.quantize(W, R, l, outer=outer)
    for key in ("A", "Q", "G", "B"):
        L[key] = synth.round_to_dtype(L[key], "f16")
    L["env_dtype"] = "f16"
    T = 5 if variant == "tokens" else 1
    X = synth.make_activations(cols, T, seed=77 + outer, x_dtype="f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32", precise=(variant == "precise"), block_scaled=(variant == "block_scaled"))
    assert orc.max_rel_error(got, ref) <= (TOL_PRECISE if variant == "precise" else TOL)
    # the layer does stand for W: its product is far closer to W x than W x is to zero
    assert orc.max_rel_error(ref, X.astype(np.float64) @ W.T) < 0.9


# ---------------------------------------------------------------- a tall, ragged projection (vocabulary-sized)
@pytest.mark.parametrize("T,variant", [(1, "auto"), (1, "block_scaled"), (3, "auto"), (70, "auto")])
def test_tall_ragged_projection(gpu, T, variant):
    """m = 32003 rows (2001 row tiles: 31 full groups of the packed layout and a ragged one), k = 1000
    (not a multiple of 128).  Every output is checked: the factored oracle is cheap at this shape."""
    L = synth.make_layer(32003, 1536, 1000, 16, seed=321, env_dtype="f16", env_kind="llama", signed_env=True)
    X = synth.make_activations(1536, T, seed=322, x_dtype="f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, "f16", "f32", block_scaled=(variant == "block_scaled"))
    assert got.shape == (T, 32003)
    assert orc.max_rel_error(got, ref) <= TOL


def test_sibling_projections_share_their_input(gpu):
    """q, k, v (and gate, up) of a decoder layer read the same activations: three layers of one plan point
    at one X buffer; each result equals the oracle's for that layer."""
    torch, mb = gpu
    X = synth.make_activations(1024, 1, seed=901, x_dtype="f16")
    Xd = _to_dev(torch, X, "f16")
    layers, Ys, refs = [], [], []
    for i, (m, k) in enumerate([(1024, 640), (1024, 640), (512, 384)]):
        L = synth.make_layer(m, 1024, k, 16, seed=910 + i, env_dtype="f16", env_kind="llama", signed_env=True)
        layers.append(mb.DeviceLayer.from_host(L))
        Ys.append(torch.zeros((1, m), dtype=torch.float32, device="cuda:0"))
        refs.append(orc.forward_factored(*_oracle_args(L), X))
    plan = mb.BatchPlan(layers, [Xd, Xd, Xd], Ys)
    plan.run()
    torch.cuda.synchronize()
    for Yb, ref in zip(Ys, refs):
        assert orc.max_rel_error(Yb.cpu().numpy(), ref) <= TOL


# ---------------------------------------------------------------- small envelope ranks through zero modes
@pytest.mark.parametrize("l,l_to,T", [(1, 8, 1), (3, 8, 1), (2, 16, 1), (3, 8, 5)])
def test_padded_envelopes_denote_the_same_layer(gpu, l, l_to, T):
    """mdbf_pad_envelope appends zero modes: bit-exact copy plus zeros, and the padded layer (which the
    matrix-core kernels take) gives the product of the original one."""
    torch, mb = gpu
    L = synth.make_layer(530, 2100, 1100, l, seed=400 + l, env_dtype="f16", env_kind="llama", signed_env=True)
    dl = mb.DeviceLayer.from_host(L)
    dp = dl.padded(l_to)
    for name in ("A", "Q", "G", "B"):
        src, dst = getattr(dl, name).cpu().numpy(), getattr(dp, name).cpu().numpy()
        assert dst.shape == (src.shape[0], l_to)
        np.testing.assert_array_equal(dst[:, :l].view(np.uint16), src.view(np.uint16))
        assert not dst[:, l:].view(np.uint16).any()
    X = synth.make_activations(2100, T, seed=410, x_dtype="f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    Xd = _to_dev(torch, X, "f16")
    for layer, bs in ((dl, False), (dp, False), (dp, True)):
        Y = mb.mdbf_forward(layer, Xd, y_dtype="f32", block_scaled=bs)
        torch.cuda.synchronize()
        assert orc.max_rel_error(Y.cpu().numpy().astype(np.float64), ref) <= TOL


# ---------------------------------------------------------------- the matrix itself, through unit vectors
@pytest.mark.parametrize("l,env_dtype", [(16, "f16"), (8, "f16"), (3, "f32")])
def test_forward_on_the_identity_reproduces_the_dense_matrix(gpu, l, env_dtype):
    """The product applied to the n unit vectors is What itself (Eq. "me-dbf-basis"), entry by entry."""
    torch, mb = gpu
    m, n, k = 200, 192, 96
    L = synth.make_layer(m, n, k, l, seed=777 + l, env_dtype=env_dtype, env_kind="unit", signed_env=True)
    W = orc.dense_reconstruct(*_oracle_args(L))
    got = _run(gpu, L, np.eye(n), "f16", "f32")              # (n, m): row j = What e_j
    assert np.abs(got.T - W).max() <= TOL * np.abs(W).max()
    one = _run(gpu, L, np.eye(n)[5:6], "f16", "f32")          # a single unit vector takes the one-token kernels
    assert np.abs(one[0] - W[:, 5]).max() <= TOL * np.abs(W).max()


# ---------------------------------------------------------------- single short calls: the split-K variant
@pytest.mark.parametrize("m,n,k,l,T,x_dtype", [
    (16, 8, 8, 16, 2, "f16"),            # one block, three of the four waves idle
    (300, 1160, 648, 16, 7, "f16"),      # 10 and 6 column blocks: partial last iterations
    (2064, 520, 4104, 16, 16, "bf16"),
    (530, 2104, 1096, 8, 3, "f32"),
    (4096, 4096, 2656, 16, 16, "f16"),
])
def test_short_single_calls(gpu, m, n, k, l, T, x_dtype):
    L = synth.make_layer(m, n, k, l, seed=m + n + k + T, env_dtype="f16", env_kind="unit", signed_env=True)
    X = synth.make_activations(n, T, seed=55 + T, x_dtype=x_dtype)
    ref = orc.forward_factored(*_oracle_args(L), X)
    got = _run(gpu, L, X, x_dtype, "f32")
    assert orc.max_rel_error(got, ref) <= TOL
    again = _run(gpu, L, X, x_dtype, "f32")
    np.testing.assert_array_equal(got, again)     # the partial sums are added in a fixed order


# ---------------------------------------------------------------- HIP graph capture and replay
@pytest.mark.parametrize("T,block_scaled", [(1, False), (1, True), (6, False)])
def test_graph_replay_matches_eager(gpu, T, block_scaled):
    """A plan captured into a HIP graph: every replay, with new activations in the same buffers and eager
    work in between, gives exactly what the eager call gives (the library records kernel launches only)."""
    torch, mb = gpu
    specs = [(530, 2104, 1104, 16), (272, 1032, 4096, 16), (1024, 1024, 640, 8)]
    layers, Xs, Ys = [], [], []
    for i, (m, n, k, l) in enumerate(specs):
        L = synth.make_layer(m, n, k, l, seed=600 + i, env_dtype="f16", env_kind="llama", signed_env=True)
        layers.append(mb.DeviceLayer.from_host(L))
        Xs.append(torch.zeros((T, n), dtype=torch.float16, device="cuda:0"))
        Ys.append(torch.zeros((T, m), dtype=torch.float32, device="cuda:0"))
    plan = mb.BatchPlan(layers, Xs, Ys, block_scaled=block_scaled)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        plan.run(stream=s)                       # warm-up outside the capture (function attributes)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        plan.run(stream=s)
    for rep in range(3):
        new = [synth.make_activations(X.shape[1], T, seed=700 + 10 * rep + i, x_dtype="f16") for i, X in enumerate(Xs)]
        for X, a in zip(Xs, new):
            X.copy_(_to_dev(torch, a, "f16"))
        for Y in Ys:
            Y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        replayed = [Y.clone() for Y in Ys]
        for Y in Ys:
            Y.zero_()
        plan.run()
        torch.cuda.synchronize()
        for Yr, Ye in zip(replayed, Ys):
            assert torch.equal(Yr, Ye)
            assert Ye.abs().max().item() > 0


# ---------------------------------------------------------------- a residual stack as one launch
@pytest.mark.parametrize("ranks,T", [((4, 4), 1), ((8, 8), 1), ((1, 1), 1), ((8, 8), 6)])
def test_residual_stack_as_one_concatenated_layer(gpu, ranks, T):
    """P independently factorised terms with sum of ranks <= 16, written as one layer (sign bases
    concatenated along the inner dimension, block-diagonal inner envelope factors): one call instead of P
    accumulating ones; ranks adding up to 8 or 16 take the matrix-core kernels."""
    terms = [synth.make_layer(530, 1032, 520 + 8 * p, l, seed=820 + p, env_dtype="f16", env_kind="llama", signed_env=True)
             for p, l in enumerate(ranks)]
    X = synth.make_activations(1032, T, seed=830, x_dtype="f16")
    ref = orc.forward_residual_stack([_oracle_args(t) for t in terms], X)
    one = concat_terms(terms)
    assert orc.max_rel_error(_run(gpu, one, X, "f16", "f32"), ref) <= TOL
    if sum(ranks) in (8, 16) and T == 1:
        assert orc.max_rel_error(_run(gpu, one, X, "f16", "f32", block_scaled=True), ref) <= TOL


# ---------------------------------------------------------------- magnitudes far from one
@pytest.mark.parametrize("env_scale,x_scale", [(0.5, 1.0), (32.0, 2.0 ** -10), (1.0, 512.0), (4.0, 2.0 ** -4), (0.25, 1.0),
                                               (0.5, 2.0 ** -6)])
@pytest.mark.parametrize("variant", ["auto", "block_scaled", "tokens"])
def test_relative_error_does_not_depend_on_scale(gpu, env_scale, x_scale, variant):
    """Envelopes and activations scaled by powers of two, the scaled activations B o x and Q o z (divided by
    8 in the fp16 variant's staging) staying inside fp16's normal range: the error relative to the largest
    output stays within the gate in every variant."""
    L = synth.make_layer(530, 2104, 1104, 16, seed=941, env_dtype="f16", env_kind="llama", signed_env=True)
    for key in ("A", "Q", "G", "B"):
        L[key] = synth.round_to_dtype(L[key].astype(np.float64) * env_scale, "f16")
    T = 5 if variant == "tokens" else 1
    X = synth.round_to_dtype(synth.make_activations(2104, T, seed=942, x_dtype="f32").astype(np.float64) * x_scale, "f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    assert np.isfinite(ref).all() and np.abs(ref).max() > 0
    got = _run(gpu, L, X, "f16", "f32", block_scaled=(variant == "block_scaled"))
    assert orc.max_rel_error(got, ref) <= TOL


@pytest.mark.parametrize("env_scale,x_scale", [(2.0 ** -9, 1.0), (2.0 ** -6, 2.0 ** -12), (2.0 ** -3, 2.0 ** -14)])
@pytest.mark.parametrize("block_scaled", [True, False])
def test_one_token_variants_carry_their_own_exponents(gpu, env_scale, x_scale, block_scaled):
    """Far below fp16's normal range (the scaled activations Q o z reach 1e-12 here) both one-token variants
    still meet the gate: the block-scaled records hold an exponent per 32 values, the fp16 variant's
    scale-in kernel one per 1024 columns, and z stays in fp32."""
    L = synth.make_layer(530, 2104, 1104, 16, seed=941, env_dtype="f16", env_kind="llama", signed_env=True)
    for key in ("A", "Q", "G", "B"):
        L[key] = synth.round_to_dtype(L[key].astype(np.float64) * env_scale, "f16")
    X = synth.round_to_dtype(synth.make_activations(2104, 1, seed=942, x_dtype="f32").astype(np.float64) * x_scale, "f16")
    ref = orc.forward_factored(*_oracle_args(L), X)
    assert np.abs(ref).max() > 0
    got = _run(gpu, L, X, "f16", "f32", block_scaled=block_scaled)
    assert orc.max_rel_error(got, ref) <= TOL
