// Host side of a call from Python: checks the tensors, fills in the C ABI's arguments, allocates what
// the caller did not bring and calls the library, in one step.
//
// A call on a small batch takes the GPU 5 to 10 us; marshalling it in Python took the host 12 us
// (attribute look-ups, shape tuples, ctypes conversions, a stream object: 16 x 256 tokens through
// BleuScorer), 21 us with outputs and workspace to allocate (rouge_n) and 37 us for a one-shot
// corpus score (which also filled two tensors and copied one on the GPU).  Here these take 3.6, 5.7
// and 7.8 us, of which 2.3 are each kernel's launch.
//
// Every function returns None for whatever is not the plain case -- tensors that are not contiguous or
// of another type, wrong shapes, a status other than TB_OK.  Up to then it has written nothing but
// token_bytes, ref_rows and ref_count of the caller's config, which the general way that the caller then
// takes sets again; that way converts, or raises the error that says what is wrong.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>

#include "tensorbleu.h"

namespace {

enum Entry { kSentence = 0, kCorpus = 1 };

struct Names {
  PyObject *clipped, *total, *closest_ref_len, *group_distinct, *corpus_stats, *device_status;
  PyObject *ref_offsets_tensor, *max_refs;
} names;

const at::Tensor* tensor(PyObject* o) {
  return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr;
}
bool plain(const at::Tensor* t, int dims, at::ScalarType type) {
  return t && t->is_cuda() && t->layout() == at::kStrided && t->dim() == dims &&
         t->scalar_type() == type && t->is_contiguous();
}
at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
  return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}
at::ScalarType score_type(const tb_config_t& cfg) {
  return cfg.score_bytes == 2 ? at::kBFloat16 : at::kFloat;
}

struct Batch {
  const at::Tensor *cand, *cand_len, *refs, *ref_len;
  int64_t B, R, cand_stride, ref_stride;
};

// cfg_object: the Python object that holds the tensor behind cfg->ref_offsets, or null
bool take_batch(PyObject* const* args, tb_config_t* cfg, PyObject* cfg_object, Batch* b) {
  b->cand = tensor(args[0]);
  b->cand_len = tensor(args[1]);
  b->refs = tensor(args[2]);
  b->ref_len = tensor(args[3]);
  if (!b->cand) return false;
  const at::ScalarType ids = b->cand->scalar_type();
  if (ids != at::kInt && ids != at::kLong) return false;
  const bool lists = cfg->ref_offsets != nullptr;
  if (!plain(b->cand, 2, ids) || !plain(b->refs, lists ? 2 : 3, ids) ||
      !plain(b->cand_len, 1, at::kInt) || !plain(b->ref_len, lists ? 1 : 2, at::kInt))
    return false;
  b->B = b->cand->size(0);
  b->cand_stride = b->cand->size(1);
  if (b->B < 1 || b->B > INT32_MAX || b->cand_len->size(0) != b->B) return false;
  int64_t rows = 0;
  if (lists) {
    if (!cfg_object) return false;
    rows = b->refs->size(0);
    b->ref_stride = b->refs->size(1);
    PyObject* offsets = PyObject_GetAttr(cfg_object, names.ref_offsets_tensor);
    PyObject* most = PyObject_GetAttr(cfg_object, names.max_refs);
    const at::Tensor* t = offsets ? tensor(offsets) : nullptr;
    const bool fits = t && t->numel() == b->B + 1 && b->ref_len->size(0) == rows;
    b->R = most ? PyLong_AsLong(most) : -1;
    Py_XDECREF(offsets);
    Py_XDECREF(most);
    PyErr_Clear();
    if (!fits) return false;
  } else {
    b->R = b->refs->size(1);
    b->ref_stride = b->refs->size(2);
    if (b->refs->size(0) != b->B || b->ref_len->size(0) != b->B || b->ref_len->size(1) != b->R)
      return false;
  }
  if (b->R < 1 || b->R > INT32_MAX) return false;
  cfg->token_bytes = ids == at::kLong ? 8 : 4;
  if (lists) cfg->ref_rows = rows;
  return true;
}

// a Stats object's tensors; false: one of them is none of ours
bool take_stats(PyObject* o, tb_stats_t* s) {
  struct { PyObject* name; void** to; } fields[] = {
      {names.clipped, reinterpret_cast<void**>(&s->clipped)},
      {names.total, reinterpret_cast<void**>(&s->total)},
      {names.closest_ref_len, reinterpret_cast<void**>(&s->closest_ref_len)},
      {names.group_distinct, reinterpret_cast<void**>(&s->group_distinct)},
      {names.corpus_stats, reinterpret_cast<void**>(&s->corpus_stats)},
      {names.device_status, reinterpret_cast<void**>(&s->device_status)}};
  for (auto& f : fields) {
    PyObject* v = PyObject_GetAttr(o, f.name);
    if (!v) {
      PyErr_Clear();
      return false;
    }
    const bool none = v == Py_None;
    const at::Tensor* t = none ? nullptr : tensor(v);
    *f.to = t ? t->data_ptr() : nullptr;
    Py_DECREF(v);  // (the object keeps it)
    if (!none && !t) return false;
  }
  return true;
}

struct Config {  // the ctypes structure's memory
  Py_buffer view;
  tb_config_t* p = nullptr;
  explicit Config(PyObject* o) {
    if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE) != 0) {
      PyErr_Clear();
      return;
    }
    if (view.len == Py_ssize_t(sizeof(tb_config_t)))
      p = static_cast<tb_config_t*>(view.buf);
    else
      PyBuffer_Release(&view);
  }
  ~Config() {
    if (p) PyBuffer_Release(&view);
  }
};

int run(Entry entry, const Batch& b, const tb_config_t* cfg, void* out, const tb_stats_t* stats,
        void* workspace, size_t bytes) {
  void* stream = static_cast<void*>(c10::hip::getCurrentHIPStream().stream());
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = (entry == kCorpus ? tensorbleu_corpus : tensorbleu_sentence)(
      b.cand->data_ptr(), b.cand_stride, b.cand_len->data_ptr<int32_t>(), b.refs->data_ptr(),
      b.ref_stride, b.ref_len->data_ptr<int32_t>(), int32_t(b.B), int32_t(b.R), cfg, out, stats,
      workspace, bytes, stream);
  Py_END_ALLOW_THREADS
  return rc;
}

at::Tensor make_workspace(const Batch& b, const tb_config_t& cfg) {
  const size_t bytes = tensorbleu_workspace_bytes(int32_t(b.B), int32_t(b.R), b.cand_stride,
                                                  b.ref_stride, &cfg);
  return bytes ? make({int64_t(bytes)}, at::kByte, *b.cand) : at::Tensor();
}

// bleu(corpus, cand, cand_len, refs, ref_len, cfg, out, stats, workspace): out or None
// bleu(..., shape, ref_count): for a scorer built for shape = (B, R, cand_stride, ref_stride);
// cfg's ref_count then is the tensor given here, or none
PyObject* bleu(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 9 && n != 11) Py_RETURN_NONE;
  Config cfg(args[5]);
  Batch b;
  tb_stats_t stats;
  if (!cfg.p) Py_RETURN_NONE;
  const Entry entry = args[0] == Py_True ? kCorpus : kSentence;
  const int32_t* ref_count = nullptr;
  if (n == 11 && args[10] != Py_None) {
    const at::Tensor* t = tensor(args[10]);
    if (!plain(t, 1, at::kInt)) Py_RETURN_NONE;
    ref_count = t->data_ptr<int32_t>();
  }
  if (!take_batch(args + 1, cfg.p, n == 9 ? args[5] : nullptr, &b)) Py_RETURN_NONE;
  if (n == 11) {
    if (!PyTuple_CheckExact(args[9]) || PyTuple_GET_SIZE(args[9]) != 4) Py_RETURN_NONE;
    const int64_t is[4] = {b.B, b.R, b.cand_stride, b.ref_stride};
    for (int i = 0; i < 4; ++i)
      if (PyLong_AsLong(PyTuple_GET_ITEM(args[9], i)) != is[i]) {
        PyErr_Clear();
        Py_RETURN_NONE;
      }
    if (ref_count && tensor(args[10])->size(0) != b.B) Py_RETURN_NONE;
    cfg.p->ref_count = ref_count;
  }
  if (args[7] != Py_None && !take_stats(args[7], &stats)) Py_RETURN_NONE;
  at::Tensor out, workspace;
  if (args[6] == Py_None) {
    out = make({entry == kCorpus ? 1 : b.B}, score_type(*cfg.p), *b.cand);
  } else {
    const at::Tensor* t = tensor(args[6]);
    if (!plain(t, 1, score_type(*cfg.p)) || t->size(0) != (entry == kCorpus ? 1 : b.B))
      Py_RETURN_NONE;
    out = *t;
  }
  if (args[8] == Py_None) {
    workspace = make_workspace(b, *cfg.p);
    if (!workspace.defined()) Py_RETURN_NONE;
  } else {
    const at::Tensor* t = tensor(args[8]);
    if (!t) Py_RETURN_NONE;
    workspace = *t;
  }
  if (run(entry, b, cfg.p, out.data_ptr(), args[7] == Py_None ? nullptr : &stats,
          workspace.data_ptr(), size_t(workspace.numel())) != TB_OK)
    Py_RETURN_NONE;
  if (args[6] != Py_None) {
    Py_INCREF(args[6]);
    return args[6];
  }
  return THPVariable_Wrap(std::move(out));
}

bool take_int(PyObject* o, int32_t* to) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  *to = int32_t(v);
  return !overflow && v == *to;
}
bool take_float(PyObject* o, float* to) {
  if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
  const double v = PyFloat_AsDouble(o);
  if (PyErr_Occurred()) {  // an integer beyond a double's range
    PyErr_Clear();
    return false;
  }
  *to = float(v);
  return true;
}

// once(corpus, cand, cand_len, refs, ref_len, max_n, smoothing, smooth_param, vocab_size,
// bfloat16): a new score tensor or None
PyObject* once(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 10) Py_RETURN_NONE;
  const Entry entry = args[0] == Py_True ? kCorpus : kSentence;
  tb_config_t cfg = {};
  if (!take_int(args[5], &cfg.max_n) || !take_int(args[6], &cfg.smoothing) ||
      !take_float(args[7], &cfg.smooth_param) || !take_int(args[8], &cfg.vocab_size))
    Py_RETURN_NONE;
  cfg.score_bytes = args[9] == Py_True ? 2 : 4;
  Batch b;
  if (!take_batch(args + 1, &cfg, nullptr, &b)) Py_RETURN_NONE;
  at::Tensor workspace = make_workspace(b, cfg);
  if (!workspace.defined()) Py_RETURN_NONE;
  at::Tensor out = make({entry == kCorpus ? 1 : b.B}, score_type(cfg), *b.cand);
  if (run(entry, b, &cfg, out.data_ptr(), nullptr, workspace.data_ptr(),
          size_t(workspace.numel())) != TB_OK)
    Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
}

// rouge(cand, cand_len, refs, ref_len, n, beta, vocab_size, ref_count, bfloat16): [B, 3] or None
PyObject* rouge(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 9) Py_RETURN_NONE;
  tb_config_t cfg = {};
  if (!take_int(args[4], &cfg.max_n) || !take_float(args[5], &cfg.smooth_param) ||
      !take_int(args[6], &cfg.vocab_size))
    Py_RETURN_NONE;
  cfg.score_bytes = args[8] == Py_True ? 2 : 4;
  Batch b;
  if (!take_batch(args, &cfg, nullptr, &b)) Py_RETURN_NONE;
  if (args[7] != Py_None) {
    const at::Tensor* t = tensor(args[7]);
    if (!plain(t, 1, at::kInt) || t->size(0) != b.B) Py_RETURN_NONE;
    cfg.ref_count = t->data_ptr<int32_t>();
  }
  tb_layout_t layout;
  if (tensorbleu_workspace_layout(int32_t(b.B), int32_t(b.R), b.cand_stride, b.ref_stride, &cfg,
                                  &layout) != TB_OK)
    Py_RETURN_NONE;
  if (layout.path == TB_PATH_GLOBAL && !layout.global_candidate_first &&
      !layout.global_partitions && !layout.global_tables_in_hbm)
    Py_RETURN_NONE;
  at::Tensor workspace = make({int64_t(layout.bytes)}, at::kByte, *b.cand);
  at::Tensor out = make({b.B, 3}, score_type(cfg), *b.cand);
  void* stream = static_cast<void*>(c10::hip::getCurrentHIPStream().stream());
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = tensorrouge_n(b.cand->data_ptr(), b.cand_stride, b.cand_len->data_ptr<int32_t>(),
                     b.refs->data_ptr(), b.ref_stride, b.ref_len->data_ptr<int32_t>(),
                     int32_t(b.B), int32_t(b.R), &cfg, out.data_ptr(), nullptr, nullptr, nullptr,
                     workspace.data_ptr(), layout.bytes, stream);
  Py_END_ALLOW_THREADS
  if (rc != TB_OK) Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
}

// at:: functions throw (out of memory): to Python as the exceptions that torch itself raises
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return F(self, args, n);
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"bleu", reinterpret_cast<PyCFunction>(guarded<bleu>), METH_FASTCALL, nullptr},
    {"once", reinterpret_cast<PyCFunction>(guarded<once>), METH_FASTCALL, nullptr},
    {"rouge", reinterpret_cast<PyCFunction>(guarded<rouge>), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) {
  names.clipped = PyUnicode_InternFromString("clipped");
  names.total = PyUnicode_InternFromString("total");
  names.closest_ref_len = PyUnicode_InternFromString("closest_ref_len");
  names.group_distinct = PyUnicode_InternFromString("group_distinct");
  names.corpus_stats = PyUnicode_InternFromString("corpus_stats");
  names.device_status = PyUnicode_InternFromString("device_status");
  names.ref_offsets_tensor = PyUnicode_InternFromString("_ref_offsets_tensor");
  names.max_refs = PyUnicode_InternFromString("_max_refs");
  return PyModule_Create(&module);
}
