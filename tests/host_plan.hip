// The planning functions of the library (sizes, launch shapes: host code without a device)
// behind a C interface. Handles are made by hand, for a chip of 256 compute units.
#include "../paper_2506_07430_amd/csrc/api.cpp"

extern "C" {

elocal_t host_handle(int n, int na, int nb) {
  elocal_ctx* h = new elocal_ctx();
  h->sys = build_sys(n, na, nb);
  return h;
}

void host_free(elocal_t h) { delete h; }

// 1 if an evaluation takes the prefix-shared kernels.
int host_prefix(elocal_t h, const elocal_ansatz* a) {
  AnsatzGeom G;
  return make_eval_geom(h, a, G) == ELOCAL_OK ? (int)G.prefix : -1;
}

// Work items of an evaluation; the tickets its launch hands out, samples per ticket's step, items
// per sample, and waves.
int64_t host_items(elocal_t h, const elocal_ansatz* a, int64_t B, int64_t* out) {
  AnsatzGeom G;
  if (make_eval_geom(h, a, G) != ELOCAL_OK) return -1;
  const EvalPlan p = plan_eval(h, G, B);
  out[0] = p.px.tickets;
  out[1] = p.px.bt;
  out[2] = p.ips;
  out[3] = p.prefix ? (int64_t)p.grid * p.waves : 0;
  return p.n_items;
}

// List-entry groups per work item of a BF16 evaluation that runs its items in parts, else 0.
int host_parts(elocal_t h, const elocal_ansatz* a, int64_t B) {
  AnsatzGeom G;
  return make_eval_geom(h, a, G) == ELOCAL_OK ? (int)plan_eval(h, G, B).parts : -1;
}

// Samples per launch of an evaluation within `bytes` (0: none), and the blocks of a launch.
int64_t host_part(elocal_t h, const elocal_ansatz* a, int64_t B, size_t bytes, int64_t* grid) {
  AnsatzGeom G;
  EvalPlan p;
  if (make_eval_geom(h, a, G) != ELOCAL_OK) return -1;
  const int64_t part = eval_part(h, G, B, bytes, p);
  *grid = part ? p.grid : 0;
  return part && eval_bytes(h, G, p, part) > bytes ? -1 : part;
}

// Bytes of the plain kernels' layout with one partial sum per item, what an evaluation needed
// before there were checkpoints or parts of items.
size_t host_plain_bytes(elocal_t h, const elocal_ansatz* a, int64_t B) {
  AnsatzGeom G;
  if (make_geom(h, a, G) != ELOCAL_OK) return 0;
  return eval_bytes(h, G, plan_eval(h, G, B, -1, 1.0, false), B);
}

// 1 if an evaluation (pauli > 0: of that many Pauli masks) finds a plan within `bytes`.
int host_fits(elocal_t h, const elocal_ansatz* a, int64_t B, size_t bytes, int64_t pauli) {
  AnsatzGeom G;
  EvalPlan p;
  if ((pauli ? make_geom(h, a, G) : make_eval_geom(h, a, G)) != ELOCAL_OK) return -1;
  return fit_plan(h, G, B, bytes, p, pauli ? pauli : -1) && eval_bytes(h, G, p, B) <= bytes;
}

// Bytes that the plan of an evaluation takes with room for all of it.
size_t host_plan_bytes(elocal_t h, const elocal_ansatz* a, int64_t B, int64_t pauli) {
  AnsatzGeom G;
  if ((pauli ? make_geom(h, a, G) : make_eval_geom(h, a, G)) != ELOCAL_OK) return 0;
  return eval_bytes(h, G, plan_eval(h, G, B, pauli ? pauli : -1), B);
}

void host_set_pauli(elocal_t h, int64_t masks) { h->pl_len = masks; }

// 1 if H on sector vectors is formed by matrix products.
int host_sector_product(elocal_t h) {
  auto choose = [](int n, int k) {
    double c = 1.0;
    for (int i = 0; i < k; ++i) c = c * (n - i) / (i + 1);
    return (int64_t)(c + 0.5);
  };
  SectorTables T;
  h->sector_nb = (uint32_t)choose(h->sys.n, h->sys.nb);
  h->sector_dim = choose(h->sys.n, h->sys.na) * h->sector_nb;
  return sector_product(h, T);
}

int host_units_le(int n, int w, int D) { return units_le(n, w, D); }

}  // extern "C"
