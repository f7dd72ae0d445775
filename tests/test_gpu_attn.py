"""GPU parity: pit_sparse_attn vs the fp64 masked-softmax oracle."""
import numpy as np
import pytest
import torch

from oracle import pit_oracle as orc
from paper_2301_10936_amd import workloads as wl
from tests.gpu_util import assert_close, bf16_bits, dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pit():
    from paper_2301_10936_amd import pit as p
    return p


def _run(pit, w, mask=None, o_dtype=torch.float32, sentinel=None):
    mask = w.mask if mask is None else mask
    out = None
    if sentinel is not None:
        out = torch.full(w.Q.shape, sentinel, dtype=o_dtype, device=dev())
    O = pit.pit_sparse_attn(to_dev(w.Q), to_dev(w.K), to_dev(w.V), to_dev(mask), w.scale, out=out, o_dtype=o_dtype)
    torch.cuda.synchronize()
    return O


@pytest.mark.parametrize("H,S,window,density", [(1, 32, 8, 0.2), (2, 64, 16, 0.1), (3, 160, 32, 0.3), (2, 512, 64, 0.05), (1, 1024, 256, 0.05)])
def test_against_oracle(pit, H, S, window, density):
    w = wl.sparse_attn(H=H, S=S, window=window, density=density, seed=S + H)
    O = _run(pit, w, sentinel=9.0)
    assert_close(O, orc.sparse_attn(w.Q, w.K, w.V, w.mask, w.scale), "sparse_attn")


def test_full_mask_is_dense_attention(pit):
    w = wl.sparse_attn(H=2, S=256, seed=3)
    full = np.ones((256, 256), dtype=np.uint8)
    O = _run(pit, w, mask=full)
    assert_close(O, orc.sparse_attn(w.Q, w.K, w.V, full, w.scale), "full mask")


def test_element_mask_inside_kept_microtiles(pit):
    """A key column kept for a single query of a block must not leak to the block's other 31 queries."""
    w = wl.sparse_attn(H=1, S=128, window=2, density=0.0, seed=4)
    m = w.mask.copy()
    m[5, 100] = 1
    m[40, 3] = 1
    m[70, :] = 0            # a query with no key at all
    O = _run(pit, w, mask=m, sentinel=4.0)
    ref = orc.sparse_attn(w.Q, w.K, w.V, m, w.scale)
    assert_close(O, ref, "element mask")
    assert torch.count_nonzero(O[0, 70]) == 0


def test_single_key_per_query_copies_value_rows(pit):
    w = wl.sparse_attn(H=2, S=96, seed=5)
    m = np.zeros((96, 96), dtype=np.uint8)
    tgt = (np.arange(96) * 7) % 96
    m[np.arange(96), tgt] = 1
    O = _run(pit, w, mask=m).cpu().numpy()
    V = orc.to_f64(w.V)
    assert np.array_equal(O, V[:, tgt])     # P = 1 exactly and bf16 V enters the product unchanged


def test_all_masked_gives_zeros(pit):
    w = wl.sparse_attn(H=1, S=64, seed=6)
    O = _run(pit, w, mask=np.zeros((64, 64), dtype=np.uint8), sentinel=2.0)
    assert torch.count_nonzero(O) == 0


def test_fp16_inputs_and_rounded_outputs(pit):
    w = wl.sparse_attn(H=2, S=256, window=32, density=0.1, seed=7)
    Q, K, V = (orc.bf16_bits_to_f64(x).astype(np.float16) for x in (w.Q, w.K, w.V))
    ref = orc.sparse_attn(Q, K, V, w.mask, w.scale)
    O = pit.pit_sparse_attn(to_dev(Q), to_dev(K), to_dev(V), to_dev(w.mask), w.scale)
    Oh = pit.pit_sparse_attn(to_dev(Q), to_dev(K), to_dev(V), to_dev(w.mask), w.scale, o_dtype=torch.float16)
    torch.cuda.synchronize()
    assert_close(O, ref, "fp16 attn")
    mx, fro = orc.rel_errors(Oh.float().cpu().numpy(), ref)
    assert fro < 1e-3 and mx < 2e-2
    wb = wl.sparse_attn(H=1, S=128, window=32, density=0.1, seed=8)
    Ob = _run(pit, wb, o_dtype=torch.bfloat16)
    mx, fro = orc.rel_errors(orc.bf16_bits_to_f64(bf16_bits(Ob)), orc.sparse_attn(wb.Q, wb.K, wb.V, wb.mask, wb.scale))
    assert fro < 3e-3   # bf16 storage costs ~1.7e-3 by itself


def test_c5_full_size(pit):
    w = wl.sparse_attn()
    O = _run(pit, w, sentinel=9.0)
    assert_close(O, orc.sparse_attn(w.Q, w.K, w.V, w.mask, w.scale), "C5 full size")


def test_attn_error_returns(pit):
    w = wl.sparse_attn(H=1, S=64, D=32, seed=1)
    with pytest.raises(pit.PitError) as e:
        _run(pit, w)
    assert e.value.code == pit.PIT_ESHAPE
    assert pit.pit_sparse_attn_workspace(1, 40, 64) == 0


def test_values_far_outside_the_fp16_range(pit):
    """bf16 V rows of magnitude 1e5 (beyond fp16's largest finite value) and 1e-9 (below its smallest
    subnormal) must come through: V enters the second product as bf16, not through a narrower type."""
    w = wl.sparse_attn(H=3, S=256, window=32, density=0.1, seed=21)
    V = orc.bf16_bits_to_f64(w.V)
    V[0] *= 1e5
    V[1] *= 1e-9
    V[2, ::2] *= 1e5          # both magnitudes among the keys of one query
    V[2, 1::2] *= 1e-9
    w.V = wl.to_bf16_bits(V.astype(np.float32))
    O = _run(pit, w, sentinel=3.0)
    assert bool(torch.isfinite(O).all())
    ref = orc.sparse_attn(w.Q, w.K, w.V, w.mask, w.scale)
    assert float(np.abs(ref[0]).max()) > 65504.0 and 0.0 < float(np.abs(ref[1]).max()) < 2.0 ** -24
    for h in range(3):
        assert_close(O[h], ref[h], f"head {h}")
    # a query that sees only tiny values: single-key mask over the 1e-9 rows of head 2 copies them exactly
    m = np.zeros((256, 256), dtype=np.uint8)
    m[np.arange(256), 1] = 1
    O1 = _run(pit, w, mask=m).cpu().numpy()
    Vq = orc.to_f64(w.V)
    assert np.array_equal(O1[2], np.broadcast_to(Vq[2, 1], (256, 64))) and np.all(O1[2, 0] != 0)


def test_key_lists_longer_than_one_pass_of_the_index_kernel(pit):
    # S = 4256: the one-launch index of the mask walks the keys in passes of 4096, so the lists of a
    # query block continue in a second pass whose last threads lie beyond the row
    w = wl.sparse_attn(H=1, S=4256, window=64, density=0.02, seed=31)
    O = _run(pit, w, sentinel=9.0)
    assert_close(O, orc.sparse_attn(w.Q, w.K, w.V, w.mask, w.scale), "sparse_attn S=4256")


def test_mask_at_an_odd_address_takes_the_general_index_build(pit):
    # a mask whose rows cannot be read 16 bytes at a time goes through pit_build_index instead of the
    # one-launch index; both must give the same attention
    w = wl.sparse_attn(H=2, S=160, window=32, density=0.2, seed=32)
    S = 160
    buf = torch.zeros(S * S + 16, dtype=torch.uint8, device=dev())
    odd = buf[3:3 + S * S].view(S, S)
    odd.copy_(to_dev(w.mask))
    assert odd.data_ptr() % 16 != 0
    Q, K, V = to_dev(w.Q), to_dev(w.K), to_dev(w.V)
    O_odd = pit.pit_sparse_attn(Q, K, V, odd, w.scale)
    O_al = pit.pit_sparse_attn(Q, K, V, to_dev(w.mask), w.scale)
    torch.cuda.synchronize()
    assert_close(O_odd, orc.sparse_attn(w.Q, w.K, w.V, w.mask, w.scale), "sparse_attn, mask at an odd address")
    assert torch.equal(O_odd, O_al)


# query blocks per compute unit on either side of each line between two and four waves per block, in heads of 8 blocks
@pytest.mark.parametrize("per_cu,more", [(3, 0), (3, 1), (4, 0), (4, 1), (5, -1), (5, 0), (6, 0), (6, 1)])
@pytest.mark.parametrize("in_dtype", [torch.bfloat16, torch.float16])
def test_two_and_four_waves_per_query_block(pit, per_cu, more, in_dtype):
    """Lists of no chunk, of fewer chunks than waves, and longer ones; all heads against the oracle (they repeat in eights), every
    output type against the four-wave kernel, and the two-wave kernel's error no larger than the four-wave kernel's."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count & ~7
    S, H = 256, per_cu * cus // 8 + more
    w = wl.sparse_attn(H=8, S=S, window=16, density=0.05, seed=H)
    m = w.mask.copy()
    m[32:96] = 0                              # a block without keys
    m[70, 5] = 1                              # .. and one with a single key
    m[128:160, :200] = 1                      # seven chunks
    q, k, v = (orc.bf16_bits_to_f64(x).astype(np.float16) if in_dtype == torch.float16 else x for x in (w.Q, w.K, w.V))
    ref = orc.sparse_attn(q, k, v, m, w.scale)
    Q, K, V = (to_dev(x).repeat(-(-H // 8), 1, 1)[:H].contiguous() for x in (q, k, v))
    run = lambda n, dt: pit.pit_sparse_attn(Q[:n].contiguous(), K[:n].contiguous(), V[:n].contiguous(), to_dev(m), w.scale, o_dtype=dt)
    O, few = run(H, torch.float32), run(8, torch.float32)                 # (8 heads: four waves)
    assert_close(O, ref[np.arange(H) % 8], "all heads")
    err = [np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) for x in (O[:8], few)]
    assert err[0] <= 1.005 * err[1]
    # the two kernels' P differ by the rounding of P (2^-17, 2^-11), their 16-bit outputs by one rounding more
    p = 2.0 ** -15 if in_dtype == torch.bfloat16 else 2.0 ** -9
    for dt, tol in ((torch.float32, p), (torch.bfloat16, p + 2.0 ** -7), (torch.float16, p + 2.0 ** -10)):
        O, few = run(H, dt).float(), run(8, dt).float()
        scale = torch.maximum(few.abs(), few.square().mean().sqrt())
        for h0 in range(0, H, 8):
            n = min(8, H - h0)
            assert float(((O[h0:h0 + n] - few[:n]).abs() / scale[:n]).max()) <= tol


def _masks(S):
    """Masks under which a query's keys take every place in a chunk of 32, or only some of them."""
    g = np.random.default_rng(S)
    i, j = np.arange(S)[:, None], np.arange(S)[None, :]
    band = (np.abs(i - j) <= 32) | np.repeat(g.random((S // 32, S)) < 0.1, 32, axis=0)
    return {"band": band, "full": np.ones((S, S), bool), "random": g.random((S, S)) < 0.2, "stride": (j - i) % 8 == 0,
            "residue": (j % 8 == 2) | ((j % 8 == 6) & (i % 2 == 0))}


@pytest.mark.parametrize("kind", ["band", "full", "random", "stride", "residue"])
@pytest.mark.parametrize("in_dtype", [torch.bfloat16, torch.float16])
def test_a_head_does_not_depend_on_the_others(pit, kind, in_dtype):
    """Two waves per query block or four, chosen by the number of heads: the same bits, whatever the mask, the output type and
    the values (with an infinity in V, too, for which the header promises nothing: with fp16 inputs it stays one at queries
    that see every key of their block)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count & ~7
    S, H = 256, 4 * cus // 8                                              # (four blocks per compute unit: two waves)
    w = wl.sparse_attn(H=4, S=S, seed=H)
    m = _masks(S)[kind].astype(np.uint8)
    q, k, v = (orc.bf16_bits_to_f64(x).astype(np.float16) if in_dtype == torch.float16 else x for x in (w.Q, w.K, w.V))
    Q, K, V = (to_dev(x) for x in (q, k, v))
    run = lambda n, V, dt: pit.pit_sparse_attn(*(x.repeat(-(-n // 4), 1, 1)[:n].contiguous() for x in (Q, K, V)), to_dev(m), w.scale, o_dtype=dt)
    V_inf = V.clone()
    V_inf[1, 10, 3], V_inf[2, 12, 40] = float("inf"), float("-inf")
    for values in (V, V_inf):
        for dt in (torch.float32, torch.bfloat16, torch.float16):
            O, few = run(H, values, dt), run(4, values, dt)
            same = O.view(-1, 4, S, 64).view(torch.uint8) == few.view(torch.uint8)
            assert bool(same.all())
    err = np.abs(run(H, V, torch.float32)[:4].cpu().numpy() - orc.sparse_attn(q, k, v, m, w.scale)).max()
    # P to 2^-17 or 2^-11 of itself, |V| < 6, and fp32 sums of up to S terms
    assert err <= 6.0 * ((2.0 ** -17 if in_dtype == torch.bfloat16 else 2.0 ** -11) + S * 2.0 ** -24)
    if in_dtype == torch.float16 and kind == "full":
        O = run(H, V_inf, torch.float32)[:4].cpu().numpy()
        assert np.all(O[1, :, 3] == np.inf) and np.all(O[2, :, 40] == -np.inf)


@pytest.mark.parametrize("scale", [-0.125, 0.0, 1e-30, 1.5])
@pytest.mark.parametrize("in_dtype", [torch.bfloat16, torch.float16])
def test_scales_and_lists_that_end_inside_a_chunk(pit, scale, in_dtype):
    """The scale is applied to differences from the largest score (a negative one through the signs of Q, zero beforehand);
    lists of 1 to 70 keys end at every kind of place in a chunk of 32, with other lists' words behind them."""
    S = 160
    w = wl.sparse_attn(H=2, S=S, seed=11)
    mask = np.zeros((S, S), dtype=np.uint8)
    for b, n in enumerate((1, 31, 33, 64, 70)):                  # keys listed by the blocks of 32 queries
        mask[32 * b:32 * (b + 1), np.random.default_rng(b).permutation(S)[:n]] = 1
    mask[40, :] = 0                                              # a query without a key
    Q, K, V = (to_dev(x).to(in_dtype) for x in (w.Q, w.K, w.V))
    O = pit.pit_sparse_attn(Q, K, V, to_dev(mask), scale)
    torch.cuda.synchronize()
    ref = orc.sparse_attn(Q.double().cpu().numpy(), K.double().cpu().numpy(), V.double().cpu().numpy(), mask, scale)
    # fp16 inputs: probabilities have 11 bits (2^-12 of each at most, so of the row); bf16 inputs: 17 bits
    tol = 2.0 ** -11 if in_dtype == torch.float16 else 2.0 ** -15
    assert np.abs(O.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.parametrize("scale", [1e-38, -1e-38])
@pytest.mark.parametrize("H,S", [(2, 64), (4, 6208)])
def test_finite_scores_whose_difference_is_not(pit, H, S, scale):
    """Scores of +-2.25e38 with a scale that leaves differences of up to 4.5 of them: the difference of two is beyond fp32.  (Blocks of
    four waves, and of two between three and four blocks per compute unit.)"""
    if S > 64 and not 3 < H * S / 32 / torch.cuda.get_device_properties(0).multi_processor_count <= 4:
        pytest.skip("sizes for 256 compute units")
    g = torch.Generator(device="cuda").manual_seed(S)
    Q, K = (torch.zeros((H, S, 64), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    Q[:, :, 9] = 1.5e19
    K[:, :, 9] = 1.5e19 * (1.0 - (torch.arange(S, device="cuda") % 9) / 4.0)
    V = torch.randn((H, S, 64), generator=g, device="cuda").to(torch.bfloat16)
    mask = torch.zeros((S, S), dtype=torch.uint8, device="cuda")
    mask[:, :64] = 1
    O = pit.pit_sparse_attn(Q, K, V, mask, scale)
    w = torch.softmax(scale * (Q[:, :1, 9].double() * K[:, :64, 9].double()), dim=1)
    ref = (w[:, :, None] * V[:, :64].double()).sum(dim=1, keepdim=True)
    assert float((O - ref).abs().max()) <= 2.0 ** -15 * float(ref.abs().max())


@pytest.mark.parametrize("scale", [-0.125, 0.0, 0.125])
@pytest.mark.parametrize("in_dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("H,S", [(2, 160), (16, 1600)])
@pytest.mark.parametrize("at", [0, 1])
def test_lists_with_set_bits_behind_their_ends(pit, H, S, in_dtype, scale, at):
    """A workspace of ones: each word that is read past the end of a list has all its bits set (a mask at an even address: a
    list per S words), or it is another list's (at an odd one: the lists side by side).  Four waves per block, and two (800 blocks
    on 256 compute units); scales that take the signs of Q and the scores scaled beforehand in both."""
    w = wl.sparse_attn(H=H, S=S, seed=11)
    mask = np.zeros((S, S), dtype=np.uint8)
    for b in range(S // 32):                                     # keys listed by the blocks of 32 queries
        keys = np.random.default_rng(b).permutation(S)[:(1, 31, 33, 64, 70)[b % 5]]
        mask[32 * b:32 * (b + 1), keys] = 1
    mask[40, :] = 0                                              # a query without a key
    mask[50, np.nonzero(mask[50])[0][1:]] = 0                    # and one with one
    Q, K, V = (to_dev(x).to(in_dtype) for x in (w.Q, w.K, w.V))
    buf = torch.zeros(S * S + 16, dtype=torch.uint8, device=dev())
    tm = buf[at:at + S * S].view(S, S)
    tm.copy_(to_dev(mask))
    ws = torch.full((pit.pit_sparse_attn_workspace(H, S, 64),), 255, dtype=torch.uint8, device=dev())
    O = pit.pit_sparse_attn(Q, K, V, tm, scale, out=torch.full((H, S, 64), 9.0, device=dev()), ws=ws)
    ref = orc.sparse_attn(Q.double().cpu().numpy(), K.double().cpu().numpy(), V.double().cpu().numpy(), mask, scale)
    # fp16 inputs: probabilities have 11 bits (2^-12 of each at most, so of the row); bf16 inputs: 17 bits
    tol = 2.0 ** -11 if in_dtype == torch.float16 else 2.0 ** -15
    assert np.abs(O.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
