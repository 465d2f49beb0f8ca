"""The surrogate-gradient form at the sizes where its kernels change form or have remainders,
against the oracle with the tolerances of test_gpu_bptt: batches that fill slices of 8 or not,
hidden sizes around the 32 neurons of an adjoint workgroup, the words of a wavefront and the
limits of the event-driven and the sliced form, step counts around a chunk, synapse rows
longer than the rounds requested ahead, more readouts than one LDS chunk or wavefront, and
spike rates at which the forward pass turns from rows to columns."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from test_gpu_bptt import _compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _inputs(B, T, C, H, O, p_in=0.4, p_rec=0.3, seed=31):
    return W.bptt_inputs(batch=B, steps=T, n_in=C, n_hidden=H, n_out=O, p_in=p_in, p_rec=p_rec, rate_lo=100.0,
                         rate_hi=400.0, seed=seed)


@pytest.mark.parametrize("B,H", [(1, 33), (8, 32), (9, 31), (17, 64), (63, 65), (64, 1)])
@pytest.mark.parametrize("smooth", [False, True])
def test_slices_and_neuron_blocks(B, H, smooth):
    _compare(_inputs(B, 20, 15, H, 4), 6, smooth=smooth)


@pytest.mark.parametrize("H", [255, 257, 512, 513, 1025])
def test_words_per_wavefront(H):
    _compare(_inputs(5, 18, 12, H, 3, p_rec=0.05), 5)


@pytest.mark.parametrize("H,p_rec", [(16, 0.9), (60, 0.5), (130, 0.6), (256, 0.3), (513, 0.12), (640, 0.12), (1024, 0.02)])
def test_synapses_per_lane_of_the_one_workgroup_adjoint(H, p_rec):
    """From one group of synapses per lane to more than the registers hold, with every number
    of lanes per neuron; an idle lane pair at 16 x 60."""
    _compare(_inputs(9, 11, 12, H, 3, p_rec=p_rec), 4)


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 15, 16, 17, 33])
def test_chunks_of_steps(T):
    _compare(_inputs(7, T, 25, 70, 3), 4)


@pytest.mark.parametrize("C", [1, 63, 64, 65, 130])
def test_input_words(C):
    _compare(_inputs(6, 12, C, 50, 3, p_in=0.9), 4)


@pytest.mark.parametrize("H,p_rec", [(40, 0.05), (150, 0.02), (700, 0.01)])
def test_many_spikes_against_short_columns(H, p_rec):
    """Inputs strong enough that most neurons spike at most steps: more sources than twice the
    longest column."""
    d = _inputs(6, 24, 20, H, 3, p_rec=p_rec)
    d["w_in"] = np.abs(d["w_in"]) * 3
    _, fw = _compare(d, 7)
    assert fw["s"].sum(axis=2).max() > 2 * d["mask_rec"].sum(axis=0).max()


def test_wide_hidden_layer_without_the_event_driven_form():
    _compare(_inputs(4, 10, 12, 2049, 2, p_rec=0.01), 4)


@pytest.mark.parametrize("T", [127, 128, 129, 300])
def test_chunks_of_event_lists(T):
    _compare(_inputs(4, T, 20, 33, 3), 25)


def test_more_events_than_a_list_holds():
    """Inputs active in most steps, on a batch that fills a wavefront: counts beyond a quarter
    of a chunk, beside inputs that stay below it."""
    d = W.bptt_inputs(batch=64, steps=140, n_in=12, n_hidden=40, n_out=3, p_in=0.5, p_rec=0.3, rate_lo=0.0,
                      rate_hi=900.0, seed=33)
    on = d["x"][:, :128].sum(axis=(0, 1))
    assert (on > 2048).any() and (on < 2048).any()
    _compare(d, 25)


def test_more_edges_per_target_than_one_pass():
    _compare(W.bptt_inputs(batch=3, steps=9, n_in=1100, n_hidden=37, n_out=2, p_in=1.0, p_rec=0.5, rate_lo=20.0,
                           rate_hi=60.0, seed=34), 4)


@pytest.mark.parametrize("O", [1, 32, 33, 70])
def test_readouts(O):
    _compare(_inputs(10, 17, 12, 40, O), 5)


def test_rows_longer_than_the_rounds_requested_ahead():
    d = _inputs(6, 15, 10, 300, 3, p_rec=0.7)
    assert d["mask_rec"].sum(axis=1).max() > 128 + 16
    _compare(d, 5)


def test_uneven_rows():
    """A neuron without outgoing recurrent synapses beside one with a full row."""
    d = _inputs(9, 25, 14, 90, 4, p_rec=0.1)
    d["mask_rec"][5], d["mask_rec"][7] = False, True
    d["mask_rec"][7, 7] = False
    rng = np.random.default_rng(3)
    d["w_rec"] = (rng.standard_normal(d["mask_rec"].shape) * 0.2).astype(np.float32) * d["mask_rec"]
    _compare(d, 8)


def test_no_recurrent_synapses():
    d = _inputs(5, 12, 10, 40, 3)
    d["mask_rec"][:] = False
    d["w_rec"][:] = 0
    _compare(d, 4)


@pytest.mark.parametrize("B,H,degree", [(64, 2080, 28), (64, 2080, 40), (9, 4096, 40), (17, 4096, 20), (17, 4096, 40), (64, 2561, 10)])
@pytest.mark.parametrize("smooth", [False, True])
def test_both_adjoints_of_large_layers(B, H, degree, smooth):
    """One, up to two and more rounds of the slices' workgroups on 256 compute units, with rows on
    both sides of the line between slices and a wavefront per neuron."""
    _compare(_inputs(B, 4, 6, H, 2, p_rec=degree / H), 3, smooth=smooth)


def test_more_neurons_than_the_sliced_adjoint_holds():
    d = _inputs(3, 6, 10, 4100, 2, p_rec=0.003)
    _compare(d, 4)
