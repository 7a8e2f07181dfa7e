/* Stands in for the HIP runtime's answers where there is no GPU: loaded in front of it, a device of so many compute units. */
int compute_units = 256;

int hipGetDevice(int *device) {
  *device = 0;
  return 0;
}
int hipDeviceGetAttribute(int *value, int attribute, int device) {
  (void)attribute; (void)device;
  *value = compute_units;
  return 0;
}
